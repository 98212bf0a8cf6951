"""Per-phase launch counts (RIPPLE_OPT_TIMING): FRONTIER counts the walks that are launches of their own."""
import pytest

import paper_2601_12347_amd as rp
from harness import make_pair, make_stream

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.4, "edge_del": 0.3, "feat": 0.3, "vadd": 0.0, "vdel": 0.0}
FRONTIER, SCATTER = 2, 3


# 2: every hop from the second on is pulled, its set marked by a walk of its own; 3: it is discovered by the launch that scatters
@pytest.mark.parametrize("mode", [2, 3])
def test_walks_inside_the_discovering_launch_are_not_counted(mode):
    print("case phase launches", mode, flush=True)
    pair, graph = make_pair(n=600, e=5000, d0=12, kind="sage_mean", widths=(12, 20, 16), seed=451)
    rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, mode)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 0)
    rp.ripple_set_option(pair.ctx, rp.OPT_TIMING, 1)
    stream = make_stream(pair, graph, MIX, 452)
    try:
        rp.ripple_get_stats(pair.ctx, reset=True)
        pieces = 0
        for bs in (5, 20, 20):
            ops, payload, _ = stream.next_batch(bs)
            res, _, _ = pair.step(ops, payload)
            pieces += res.n_sub_batches
            assert res.hop_mode[2] == mode
        st = rp.ripple_get_stats(pair.ctx)
    finally:
        pair.close()
    assert [st.launches[FRONTIER][l] for l in (1, 2)] == [pieces, pieces if mode == 2 else 0]
    assert [st.launches[SCATTER][l] for l in (1, 2)] == [pieces, pieces]
