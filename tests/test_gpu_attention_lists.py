"""Attention hops whose messages are listed by destination (k_gat_list): rows with their score behind the last column (up to 63 numbers), a lane
per column above; hubs that keep their long rows, created and deleted vertices. A bucket that runs over (the hop is then read through in-rows), and the rule that chooses."""
import numpy as np
import pytest

import paper_2601_12347_amd as rp
import ripple_inputs as ri
from harness import Pair, make_pair, make_stream

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
    modes = []
    try:
        for bs in (1, 2, 20, 3, 150, 10):
            ops, payload, _ = stream.next_batch(bs)
            res, _, _ = pair.step(ops, payload)
            print(" batch", bs, "hop modes", list(res.hop_mode[1:4]), "messages", list(res.messages[1:4]), flush=True)
            modes += [int(res.hop_mode[l]) for l in (2, 3) if res.messages[l]]
        pair.check_aggregates()
    finally:
        pair.close()
    assert modes and set(modes) == {4}


@pytest.mark.parametrize("room", ["lists", "over"])
def test_one_bucket_of_attention_messages(room):
    """300 vertices with the same two out-neighbours, which are not recomputed: 600 messages for one bucket. A large edge capacity leaves room for them, a
    small one does not, and the hop is read through in-rows."""
    print("case attention bucket", room, flush=True)
    n, k, widths = 3400, 300, (8, 12, 10)
    rng = np.random.default_rng(7)
    mid = np.arange(10, 10 + k)
    src = np.concatenate([np.zeros(k, np.int64), mid, mid, rng.integers(400, n, 600)])
    dst = np.concatenate([mid, np.full(k, 3), np.full(k, 2), rng.integers(400, n, 600)])
    keep = np.unique(src * n + dst)
    keep = keep[keep // n != keep % n]
    pair = Pair(n, n + 8, (keep // n).astype(np.uint32), (keep % n).astype(np.uint32), ri.features(n, widths[0], 372), ri.make_model("gat", widths, 371),
                edge_capacity=8_000_000 if room == "lists" else None)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2)
    rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    try:
        for b in range(3):
            res, _, _ = pair.step(np.array([(ri.OP_FEAT_UPDATE, 0, 0, 0)], np.uint32), rng.standard_normal((1, widths[0])).astype(np.float32))
            assert res.messages[2] == 3 * k and res.hop_mode[2] == (4 if room == "lists" else 0)
        pair.check_aggregates()
    finally:
        pair.close()


def test_attention_messages_are_listed_where_they_are_few():
    """The rule, left to itself: one changed vertex among 40,000 with 150 out-edges each sends 23 K messages at hop 2, less than a 64th of the edges, and 2 to 3 M
    at hop 3. The same batches with lists switched off give the same rows."""
    print("case attention lists chosen", flush=True)
    n, e, widths = 40_000, 6_000_000, (16, 24, 70, 10)
    rng = np.random.default_rng(17)
    keep = np.unique(rng.integers(0, n, e) * n + rng.integers(0, n, e))
    keep = keep[keep // n != keep % n]
    src, dst = (keep // n).astype(np.uint32), (keep % n).astype(np.uint32)
    rows = {}
    for mode in (1, 0):
        ctx = rp.ripple_init_graph(n, n, src, dst, ri.features(n, widths[0], 5))
        try:
            rp.ripple_set_option(ctx, rp.OPT_SORTED_MESSAGES, mode)
            rp.ripple_load_model(ctx, ri.make_model("gat", widths, 6))
            rp.ripple_full_infer(ctx)
            draw = np.random.default_rng(18)
            for b in range(4):
                u, v = draw.integers(0, n, 3), draw.integers(0, n, 3)
                ops = np.array([(ri.OP_FEAT_UPDATE, draw.integers(0, n), 0, 0)] + [(ri.OP_EDGE_ADD, x, y, 0) for x, y in zip(u, v)], np.uint32)
                res = rp.ripple_apply_updates(ctx, ops, draw.standard_normal((1, widths[0])).astype(np.float32))
                print(" batch", b, "hop modes", list(res.hop_mode[1:4]), "messages", list(res.messages[1:4]), flush=True)
                assert 14_500 < res.messages[2] < len(keep) // 64 < res.messages[3]
                assert list(res.hop_mode[1:4]) == [0, 4 if mode and b else 0, 0]     # (the first batch has no hint)
            rows[mode] = [rp.ripple_get_embeddings(ctx, l, widths[l], n_rows=n) for l in (2, 3)]
        finally:
            rp.ripple_destroy(ctx)
    for a, b in zip(rows[1], rows[0]):                      # four patches of three roundings each, of terms up to 1,000 times what is left of them (GAT_CANCEL)
        assert np.abs(a - b).max() <= 4 * 3 * 2.0 ** -24 * 1e3 * np.abs(b).max()
