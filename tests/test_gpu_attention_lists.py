"""Attention hops whose messages are listed by destination (k_gat_list): rows with their score behind the last column (up to 63 numbers), a lane
per column above; hubs that keep their long rows and some whose bucket runs over (the hop is then read through in-rows), created and deleted vertices."""
import pytest

import paper_2601_12347_amd as rp
from harness import make_pair, make_stream

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.35, "edge_del": 0.25, "feat": 0.25, "vadd": 0.08, "vdel": 0.07}


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("width", [1, 3, 4, 46, 47, 63, 64, 65, 130, 257, 520])
def test_listed_attention_messages(width, weighted):
    print("case listed attention", width, weighted, flush=True)
    widths = (12, 16, width, 10)
    pair, graph = make_pair(n=900, e=12000, d0=widths[0], kind="gat", widths=widths, seed=431, slack=128, weighted=weighted, top_share=0.04, edge_capacity=20000)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2)
    rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    stream = make_stream(pair, graph, MIX, 432, weighted=weighted)
    try:
        for bs in (1, 2, 20, 3, 150, 10):
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
        pair.check_aggregates()
    finally:
        pair.close()
