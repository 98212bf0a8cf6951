"""Hops whose rows have up to 64 numbers and are not packed (k_scatter_pull4 and k_scatter_list4 on rows of floats): widths around 4, 8 and
16 lanes of four columns, rows that begin at any multiple of four bytes and padded ones, pulled, discovered and listed, with weights and without."""
import pytest

import paper_2601_12347_amd as rp
from harness import make_pair, make_stream

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.35, "edge_del": 0.25, "feat": 0.25, "vadd": 0.08, "vdel": 0.07}


@pytest.mark.parametrize("way", ["pull", "discover", "list"])
@pytest.mark.parametrize("kind", ["gcn_sum", "gcn_wsum"])
@pytest.mark.parametrize("width", [1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64])
def test_rows_of_up_to_64_numbers(way, kind, width):
    """The second layer sends rows of `width` numbers as they are, the third rows of the same width that are projected first; hubs of
    some hundred in-edges (a sum of many messages), vertices with one or none."""
    print("case narrow rows", way, kind, width, flush=True)
    widths = (12, width, 2 * width + 1, width)
    pair, graph = make_pair(n=900, e=9000, d0=widths[0], kind=kind, widths=widths, seed=411, slack=128, weighted=kind == "gcn_wsum", top_share=0.03,
                            edge_capacity=16000, packed=0)
    rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, 3 if way == "discover" else 2)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2 if way == "list" else 0)
    rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    stream = make_stream(pair, graph, MIX, 412, weighted=kind == "gcn_wsum")
    seen = set()
    try:
        for b, bs in enumerate([1, 30, 200, 30]):
            ops, payload, _ = stream.next_batch(bs)
            res, _, _ = pair.step(ops, payload)
            seen |= set(res.hop_mode[2:4])
        pair.check_aggregates()
    finally:
        pair.close()
    assert {"pull": 2, "discover": 3, "list": 4}[way] in seen
