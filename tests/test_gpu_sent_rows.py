"""Project-first layers at the widths where the row stride of what vertices have sent changes: rows one behind the other, at multiples of 32 bytes, at
multiples of 64."""
import pytest

import paper_2601_12347_amd as rp
from harness import make_pair, make_stream

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.35, "edge_del": 0.25, "feat": 0.25, "vadd": 0.08, "vdel": 0.07}


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("width", [1, 2, 3, 5, 8, 9, 16, 17, 32, 33, 40, 41, 47, 64, 65, 81, 100])
def test_widths_of_sent_rows(width, deterministic):
    print("case sent rows", width, deterministic, flush=True)
    widths = (10, 2 * width + 1, width)
    pair, graph = make_pair(n=500, e=4000, d0=widths[0], kind="sage_mean", widths=widths, seed=441, deterministic=deterministic)
    stream = make_stream(pair, graph, MIX, 442)
    try:
        assert rp.ripple_get_layer_info(pair.ctx, 2)[1]     # project-first
        for bs in (1, 30, 30):
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
        pair.check_aggregates()
    finally:
        pair.close()
