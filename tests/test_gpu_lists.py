"""Hops from the list of their messages (k_frontier_list, k_scatter_list, k_scatter_list4): packed rows, buckets that take more than one
round, buckets that run over; and the weights beside the out-rows that pushed and listed messages are multiplied by. (Rows of other widths: test_gpu_updates.py, sorted messages.)"""
import numpy as np
import pytest
import torch

import paper_2601_12347_amd as rp
import ripple_inputs as ri
from harness import Pair, make_pair, make_stream
from ripple_inputs.graphs import OP_EDGE_ADD, OP_EDGE_DEL, OP_EDGE_REWEIGHT, OP_FEAT_UPDATE

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.4, "edge_del": 0.25, "feat": 0.2, "vadd": 0.08, "vdel": 0.07}


@pytest.mark.parametrize("mode", [0, 2])
@pytest.mark.parametrize("kind,widths,store", [("sage_mean", (12, 96, 47), "f32"), ("gcn_sum", (24, 88, 33), "f32"), ("gcn_sum", (24, 100, 48), "bf16"),
                                               ("sage_mean", (12, 96, 96, 40), "f32")])
def test_packed_rows_from_the_list(mode, kind, widths, store):
    print("case packed list", mode, kind, widths, store, flush=True)
    pair, graph = make_pair(n=900, e=9000, d0=widths[0], kind=kind, widths=widths, seed=361, slack=128, store=store)
    rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, mode)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2)
    rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    stream = make_stream(pair, graph, MIX, 363)
    listed = 0
    try:
        for b, bs in enumerate([1, 30, 200, 30, 300]):
            ops, payload, _ = stream.next_batch(bs)
            res, _, _ = pair.step(ops, payload)
            modes = list(res.hop_mode[1:len(widths)])
            print(" batch", b, bs, "hop modes", modes, flush=True)
            listed += modes[-1] == 4
        pair.check_aggregates()
    finally:
        pair.close()
    assert listed >= 2                                     # (automatic mode discovers the hops that send along most edges)


@pytest.mark.parametrize("room", ["rounds", "over"])
@pytest.mark.parametrize("widths", [(8, 24, 40, 6), (8, 96, 47)])
def test_one_destination_with_thousands_of_messages(room, widths):
    """3,000 vertices with one in-neighbour and the same two out-neighbours: when the in-neighbour's features change, hop 2 sends 3,000
    messages each to two sinks, in one bucket. With a large edge capacity the bucket has room for all of them and takes two rounds;
    with a small one it runs over and the hop is pulled or pushed."""
    n, k = 3400, 3000
    rng = np.random.default_rng(7)
    mid = np.arange(10, 10 + k)
    src = np.concatenate([np.zeros(k, np.int64), mid, mid, rng.integers(3100, n, 600)])
    dst = np.concatenate([mid, np.full(k, 3), np.full(k, 2), rng.integers(10, n, 600)])
    keep = np.unique(src * n + dst)
    src, dst = (keep // n).astype(np.uint32), (keep % n).astype(np.uint32)
    model = ri.make_model("gcn_sum", widths, 371)
    pair = Pair(n, n + 8, src, dst, ri.features(n, widths[0], 372), model, edge_capacity=4_000_000 if room == "rounds" else None, project_first=len(widths) == 3)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2)
    rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, 2)
    try:
        for b in range(3):
            ops = np.zeros((1, 4), np.uint32)
            ops[0] = (OP_FEAT_UPDATE, 0, 0, 0)
            res, _, _ = pair.step(ops, rng.standard_normal((1, widths[0])).astype(np.float32))
            print(" batch", b, "hop modes", list(res.hop_mode[1:len(widths)]), "messages", list(res.messages[1:len(widths)]), flush=True)
            assert res.messages[2] >= 2 * k
            assert b == 0 or res.hop_mode[2] == (4 if room == "rounds" else 2)   # (the first batch cuts its buckets without a hint)
        pair.check_aggregates()
    finally:
        pair.close()


MIXW = {"edge_add": 0.25, "edge_del": 0.2, "feat": 0.25, "vadd": 0.05, "vdel": 0.05, "reweight": 0.2}


@pytest.mark.parametrize("way", ["push", "list", "small"])
@pytest.mark.parametrize("kind,widths,store", [("gcn_wsum", (12, 96, 47), "f32"), ("sage_wsum", (75, 190, 190, 23), "f32"), ("gcn_wsum", (24, 300, 130), "f32"),
                                               ("gcn_wsum", (24, 100, 48), "bf16"), ("gcn_wsum", (17, 600, 40), "f32")])
def test_weights_along_out_rows(way, kind, widths, store):
    print("case out-row weights", way, kind, widths, store, flush=True)
    pair, graph = make_pair(n=700, e=6000, d0=widths[0], kind=kind, widths=widths, seed=381, slack=128, store=store, weighted=True, edge_capacity=7000)
    if way == "push":
        rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, 1)
    if way == "list":
        rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2)
        rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, 2)
    if way != "small":
        rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    stream = make_stream(pair, graph, MIXW, 383, weighted=True)
    seen = set()
    try:
        for b, bs in enumerate([1, 30, 200, 30, 300, 3, 3]):
            ops, payload, _ = stream.next_batch(bs)
            res, _, _ = pair.step(ops, payload)
            modes = list(res.hop_mode[1:len(widths)])
            print(" batch", b, bs, "hop modes", modes, flush=True)
            seen |= set(modes)
        pair.check_aggregates()
    finally:
        pair.close()
    assert (4 if way == "list" else 1) in seen


@pytest.mark.parametrize("gone", [1, 2, 64, 65, 200])
def test_weights_of_a_long_out_row(gone):
    """A vertex with 300 out-edges: `gone` of them deleted (every way in which a row closes its holes), some of the others given new weights,
    more added than the row has room for. Each time its features change and the messages along every edge of the row are compared."""
    n, k = 700, 300
    src = np.concatenate([np.zeros(k, np.uint32), np.arange(1, 600, dtype=np.uint32)])
    dst = np.concatenate([np.arange(10, 10 + k, dtype=np.uint32), np.arange(2, 601, dtype=np.uint32)])
    weights = ri.edge_weights(len(src), 391)
    pair = Pair(n, n + 8, src, dst, ri.features(n, 12, 392), ri.make_model("gcn_wsum", (12, 20, 6), 393), weights=weights)
    rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, 1)
    rng = np.random.default_rng(394)
    bits = lambda x: int(np.float32(x).view(np.uint32))
    feat = lambda: pair.step(np.array([(OP_FEAT_UPDATE, 0, 0, 0)], np.uint32), rng.standard_normal((1, 12)).astype(np.float32))
    out = rng.permutation(np.arange(10, 10 + k))
    try:
        print("case long out-row", gone, flush=True)
        feat()
        pair.step(np.array([(OP_EDGE_DEL, 0, v, 0) for v in out[:gone]] + [(OP_EDGE_REWEIGHT, 0, v, bits(rng.uniform(0.2, 2))) for v in out[gone:gone + 40]], np.uint32), None)
        feat()
        pair.step(np.array([(OP_EDGE_ADD, 0, v, bits(rng.uniform(0.2, 2))) for v in range(320, 640)], np.uint32), None)
        feat()
        pair.step(np.array([(OP_EDGE_REWEIGHT, 0, v, bits(rng.uniform(0.2, 2))) for v in range(400, 500)] + [(OP_EDGE_DEL, 0, v, 0) for v in range(320, 330)], np.uint32), None)
        feat()
        pair.check_aggregates()
        pair.check_graph()
    finally:
        pair.close()


def _feature(pair, rng, v):
    ops = np.array([(OP_FEAT_UPDATE, v, 0, 0)], np.uint32)
    res, _, _ = pair.step(ops, rng.standard_normal((1, pair.widths[0])).astype(np.float32))
    print(" vertex", v, "hop modes", list(res.hop_mode[1:pair.L + 1]), "messages", list(res.messages[1:pair.L + 1]), flush=True)
    return res


def test_a_bucket_that_ran_over_is_remembered():
    """Vertex 0 sends 3,580 messages to two sinks at hop 2 (their bucket has room for about 150), vertex 5 some 3,200 all over the graph. After
    vertex 0's batch hops of at least half its size are pulled without a list; after a small one lists are tried again."""
    n, rng = 3400, np.random.default_rng(17)
    mid, other = np.arange(10, 1800), np.arange(1800, 3390)
    src = np.concatenate([np.zeros(len(mid), np.int64), np.repeat(mid, 2), np.full(len(other), 5), np.repeat(other, 2), [7], [8]])
    dst = np.concatenate([mid, np.tile([2, 3], len(mid)), other, rng.integers(10, n, 2 * len(other)), [8], [9]])
    keep = np.unique(src * n + dst)
    src, dst = (keep // n).astype(np.uint32), (keep % n).astype(np.uint32)
    pair = Pair(n, n + 8, src, dst, ri.features(n, 8, 412), ri.make_model("gcn_sum", (8, 24, 40, 6), 411), project_first=False)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2)
    rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, 2)
    print("case bucket remembered", flush=True)
    try:
        big = _feature(pair, rng, 0)
        wide = _feature(pair, rng, 5)
        assert big.hop_mode[2] == 2 and wide.messages[2] >= big.messages[2] // 2
        assert wide.hop_mode[2] == 2
        small = _feature(pair, rng, 7)
        assert small.messages[2] < big.messages[2] // 2
        assert _feature(pair, rng, 5).hop_mode[2] == 4
        pair.check_aggregates()
    finally:
        pair.close()


def test_a_bucket_that_runs_over_where_the_hop_is_pushed():
    """3,000 messages of two numbers to a sink with 7,000 in-neighbours: the list has no room for them in one bucket, and a pull would read more
    than a push sends."""
    n, k, rng = 8000, 3000, np.random.default_rng(19)
    mid, more = np.arange(10, 10 + k), np.arange(3100, 7100)
    src = np.concatenate([np.zeros(k, np.int64), mid, more, rng.integers(3100, n, 24000)])
    dst = np.concatenate([mid, np.full(k, 2), np.full(len(more), 2), rng.integers(3100, n, 24000)])
    keep = np.unique(src * n + dst)
    src, dst = (keep // n).astype(np.uint32), (keep % n).astype(np.uint32)
    pair = Pair(n, n + 8, src, dst, ri.features(n, 8, 422), ri.make_model("gcn_sum", (8, 2, 6), 421), project_first=False)
    rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 2)
    rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
    print("case bucket over, pushed", flush=True)
    try:
        for _ in range(3):
            res = _feature(pair, rng, 0)
            assert res.messages[2] >= k and res.hop_mode[2] == 1
        pair.check_aggregates()
    finally:
        pair.close()


def test_no_room_for_lists_where_there_are_none():
    """Graphs of more than 2^25 vertices have no lists, and nothing is allocated for them. Two layers of one column take 70 bytes per vertex: rows,
    sums and changes 24, three lists with two prefixes each 36, list and prefix of the live vertices 8, marks and bitmaps 2. (Room for the lists
    of the smallest pool such a graph can have: 24 bytes per vertex more.)"""
    print("case memory of a large graph", flush=True)
    n_cap = (1 << 25) + 64
    src, dst = np.arange(0, 60, dtype=np.uint32), np.arange(1, 61, dtype=np.uint32)
    ctx = rp.ripple_init_graph(64, n_cap, src, dst, ri.features(64, 1, 432), edge_capacity=100_000)
    try:
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        rp.ripple_load_model(ctx, ri.make_model("gcn_sum", (1, 1, 1), 431))
        torch.cuda.synchronize()
        taken = before - torch.cuda.mem_get_info()[0]
        print("  bytes per vertex %.1f" % (taken / n_cap), flush=True)
        assert taken < 76 * n_cap
    finally:
        rp.ripple_destroy(ctx)


def test_weights_beside_the_out_rows_only_for_weighted_sums():
    """A weighted graph whose model has no weighted sum keeps the weights beside the in-rows alone: 4 bytes per entry of a pool, where weighted sums
    take 4 more and 12 for a quarter of the entries (lists of messages)."""
    src, dst, _, _ = ri.chung_lu_graph(700, 6000, 2.1, 0.03, 441)
    weights = ri.edge_weights(len(src), 442)
    free = {}
    for kind, w in (("gcn_sum", None), ("gcn_sum", weights), ("gcn_wsum", weights)):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        args = dict(edge_capacity=30_000_000)
        feats = ri.features(700, 12, 443)
        ctx = rp.ripple_init_graph(700, 700, src, dst, feats, **args) if w is None else rp.ripple_init_graph_weighted(700, 700, src, dst, w, feats, **args)
        try:
            rp.ripple_load_model(ctx, ri.make_model(kind, (12, 20, 6), 444))
            torch.cuda.synchronize()
            free[kind, w is not None] = before - torch.cuda.mem_get_info()[0]
        finally:
            rp.ripple_destroy(ctx)
    one, all_of_it = (free[k, True] - free["gcn_sum", False] for k in ("gcn_sum", "gcn_wsum"))
    print("case memory of weights", one, all_of_it, flush=True)
    assert one > 0 and abs(one / all_of_it - 4 / 11) < 0.05


@pytest.mark.parametrize("kind", ["gcn_sum", "sage_mean", "gcn_max", "gat"])
def test_new_weights_where_no_layer_uses_them(kind):
    """Accepted where the edge exists, rejected where it does not, and kept: nothing but the graph's weights changes."""
    print("case unused weights", kind, flush=True)
    pair, graph = make_pair(n=700, e=6000, d0=12, kind=kind, widths=(12, 20, 6), seed=451, slack=128, weighted=True, edge_capacity=7000)
    stream = make_stream(pair, graph, MIXW, 453, weighted=True)
    try:
        for b, bs in enumerate([1, 30, 300, 900]):
            print(" batch", b, bs, flush=True)
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
        u, v = np.divmod(np.flatnonzero(~np.isin(np.arange(700 * 700), pair.ora.edges()[0] * 700 + pair.ora.edges()[1])), 700)
        pick = np.random.default_rng(454).choice(len(u), 20, replace=False)
        res, rec, _ = pair.step(np.array([(OP_EDGE_REWEIGHT, u[i], v[i], 0x3F800000) for i in pick], np.uint32), None)
        assert res.n_applied == 0
        pair.check_graph()
    finally:
        pair.close()
