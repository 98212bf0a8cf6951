"""Small cases at the edges of what single kernels and dispatch rules take, each against the oracle."""
import numpy as np
import pytest

import paper_2601_12347_amd as rp
import ripple_inputs as ri
from harness import Pair, make_pair, make_stream

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.5, "edge_del": 0.3, "feat": 0.2, "vadd": 0.0, "vdel": 0.0}


@pytest.mark.parametrize("kind,weighted", [("gcn_sum", False), ("gcn_wsum", True), ("gcn_max", False), ("gcn_min", False)])
@pytest.mark.parametrize("edges", [0, 1, 255, 256, 257, 5000])
def test_bootstrap_sums_of_rows_that_span_runs(kind, weighted, edges):
    """The in-edge space is cut into runs: a vertex whose in-edges lie in several (vertex 0, up to 5,000 in-edges), a few
    short rows after it and vertices without any."""
    print("case runs", kind, edges, flush=True)
    n = 6000
    src = np.arange(1, edges + 1, dtype=np.uint32)
    dst = np.zeros(edges, np.uint32)
    if edges > 1000:
        src = np.concatenate([src, np.arange(100, 160, dtype=np.uint32)])
        dst = np.concatenate([dst, np.repeat(np.arange(1, 21, dtype=np.uint32), 3)])
    model = ri.make_model(kind, (7, 70, 9), 3)
    weights = ri.edge_weights(len(src), 4) if weighted else None
    pair = Pair(n, n + 5, src, dst, ri.features(n, 7, 1), model, weights=weights)
    try:
        pair.check_embeddings()
        pair.check_aggregates()
        rp.ripple_full_infer(pair.ctx)                     # a second time, over the sums of the first
        pair.check_embeddings()
    finally:
        pair.close()


@pytest.mark.parametrize("kind,widths,store", [
    ("gcn_sum", (1, 2, 3), "f32"), ("gcn_mean", (75, 190, 23), "f32"), ("sage_mean", (5, 129, 6), "f32"), ("gin_sum", (7, 9, 5), "f32"),
    ("gat", (13, 31, 3), "f32"), ("sage_mean", (3, 33, 127, 2), "bf16"), ("gcn_sum", (9, 65, 31), "bf16"), ("gin_sum", (6, 11, 5), "bf16")])
@pytest.mark.parametrize("self_cache", [True, False])
def test_rows_of_any_width(kind, widths, store, self_cache):
    """Widths that are not multiples of four: groups of four numbers are read past a row's end, written up to it."""
    print("case widths", kind, widths, store, self_cache, flush=True)
    pair, graph = make_pair(n=333, e=2000, d0=widths[0], kind=kind, widths=widths, store=store, seed=8, self_cache=self_cache)
    try:
        pair.check_embeddings()
        stream = make_stream(pair, graph, MIX, 9)
        for bs in (1, 60):
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
    finally:
        pair.close()


@pytest.mark.parametrize("kind,widths,store", [("gcn_sum", (12, 20, 8), "f32"), ("sage_mean", (16, 70, 130, 40), "f32"), ("gin_sum", (9, 24, 11), "f32"),
                                               ("sage_mean", (33, 100, 47), "f32"), ("gcn_mean", (40, 512, 257), "bf16"), ("gcn_sum", (100, 47, 64), "f32")])
@pytest.mark.parametrize("sizes", [(1, 1, 1, 2), (17, 16, 33, 60), (260, 511, 513, 512)])
def test_small_pieces_and_hops(kind, widths, store, sizes):
    """Batches small enough for the few-launch Apply step (up to 512 operations) and hops, on a graph with hubs; vertices are
    created with their edges; every batch but the first finds hints of the one before, some too small for it."""
    print("case small", kind, widths, store, sizes, flush=True)
    pair, graph = make_pair(n=3000, e=16000, d0=widths[0], kind=kind, widths=widths, store=store, seed=31, slack=400, top_share=0.06)
    mix = {"edge_add": 0.45, "edge_del": 0.3, "feat": 0.2, "vadd": 0.05, "vdel": 0.0}
    stream = make_stream(pair, graph, mix, 32)
    try:
        for b, bs in enumerate(sizes):
            print(" batch", b, bs, flush=True)
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
        pair.check_graph()
        pair.check_aggregates(tol=2e-2 if store == "bf16" else None)
    finally:
        pair.close()


def test_small_piece_at_the_edge_capacity_changes_nothing():
    print("case small capacity", flush=True)
    n, k = 200, 400
    src, dst = np.arange(k, dtype=np.uint32) % n, (np.arange(k, dtype=np.uint32) * 7 + 1 + np.arange(k, dtype=np.uint32) // n) % n
    pair = Pair(n, n + 4, src, dst.astype(np.uint32), ri.features(n, 5, 1), ri.make_model("gcn_sum", (5, 6, 4), 2), edge_capacity=k + 3)
    try:
        have = set(zip(src.tolist(), dst.tolist()))
        new = [(u, v) for u in range(20) for v in range(20) if u != v and (u, v) not in have]
        ops = np.array([(ri.OP_EDGE_ADD, u, v, 0) for u, v in new[:4]], dtype=np.uint32)
        before = pair.gpu_layer(2)
        with pytest.raises(rp.RippleError) as ei:
            rp.ripple_apply_updates(pair.ctx, ops, None)
        assert ei.value.status == rp.binding.RIPPLE_ECAPACITY
        assert np.array_equal(before, pair.gpu_layer(2))
        pair.step(ops[:3], None)
        pair.check_graph()
    finally:
        pair.close()


@pytest.mark.parametrize("kind,widths,store", [
    ("gcn_max", (8, 1, 5, 3), "f32"), ("gcn_min", (9, 64, 65, 7), "f32"), ("gcn_max", (16, 130, 270, 6), "bf16"), ("gat", (8, 1, 5, 3), "f32"),
    ("gat", (9, 16, 47, 63), "f32"), ("gat", (16, 64, 65, 7), "f32"), ("gat", (7, 130, 260, 4), "f32")])
def test_hops_cut_over_edges(kind, widths, store):
    """Max / min hops that recompute every candidate and attention hops, none of them listed: hubs of up to 1,000 in-edges
    that several runs share, vertices created with their edges, rows left without in-edges."""
    print("case cut hops", kind, widths, store, flush=True)
    pair, graph = make_pair(n=3000, e=16000, d0=widths[0], kind=kind, widths=widths, store=store, seed=51, slack=400, top_share=0.06)
    mix = {"edge_add": 0.4, "edge_del": 0.35, "feat": 0.2, "vadd": 0.05, "vdel": 0.0}
    stream = make_stream(pair, graph, mix, 52)
    try:
        rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
        for b, bs in enumerate((300, 600, 300)):           # from the second one on there are hints
            print(" batch", b, flush=True)
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
        pair.check_embeddings()
    finally:
        pair.close()


@pytest.mark.parametrize("deterministic,weighted", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("dels,adds", [(1, 0), (2, 1), (64, 0), (65, 64), (511, 2), (700, 324), (600, 425), (1500, 1300), (2999, 1990), (3000, 1500)])
def test_many_changes_of_one_row(deterministic, weighted, dels, adds):
    """Deletions and additions that all meet in vertex 0's in-row and vertex 1's out-row (3,000 entries each): few ones, a
    wavefront's worth and one more, what is put in order in LDS and one more, all entries."""
    print("case one row", deterministic, weighted, dels, adds, flush=True)
    n, k = 6000, 3000
    rng = np.random.default_rng(dels * 7 + adds)
    ids = np.arange(2, 2 + k, dtype=np.uint32)
    chain = np.arange(3999, 5999, dtype=np.uint32)         # (so that the new neighbours have something to send at every layer)
    src, dst = np.concatenate([ids, np.full(k, 1, np.uint32), chain]), np.concatenate([np.zeros(k, np.uint32), ids, chain + 1])
    weights = ri.edge_weights(len(src), 5) if weighted else None
    model = ri.make_model("gcn_wsum" if weighted else "sage_mean", (5, 9, 70, 4), 3)
    pair = Pair(n, n + 5, src, dst, ri.features(n, 5, 1), model, weights=weights, deterministic=deterministic, edge_capacity=20000)
    try:
        gone, new = rng.permutation(ids)[:dels], np.arange(4000, 4000 + adds, dtype=np.uint32)
        bits = (np.full(adds, 0.75, np.float32) if weighted else np.zeros(adds, np.float32)).view(np.uint32)
        for flip in (False, True):                         # in-row of 0, then out-row of 1
            a = [(ri.OP_EDGE_DEL, 1, x, 0) if flip else (ri.OP_EDGE_DEL, x, 0, 0) for x in gone]
            b = [(ri.OP_EDGE_ADD, 1, x, w) if flip else (ri.OP_EDGE_ADD, x, 0, w) for x, w in zip(new, bits)]
            ops = np.array(a + b, dtype=np.uint32)
            pair.step(ops[rng.permutation(len(ops))], None)
        pair.check_graph()
        pair.check_aggregates()
    finally:
        pair.close()


@pytest.mark.parametrize("deterministic", [False, True])
def test_batches_around_the_room_a_context_starts_with(deterministic):
    """Operations and feature rows are staged in memory that a context has from its start, up to 6,144 and 1,024 of them; larger
    batches bring room of their own, deleted vertices room for their edges. All sizes in turn on one context."""
    print("case staging", deterministic, flush=True)
    pair, _ = make_pair(n=7000, e=12000, d0=3, kind="sage_mean", widths=(3, 5, 2), seed=61, slack=8, deterministic=deterministic)
    rng = np.random.default_rng(62)
    try:
        for feats, dels in ((1, 0), (1024, 0), (1025, 0), (2, 3), (6143, 0), (6144, 1), (6145, 0), (3, 0)):
            print(" feature rows", feats, "deleted", dels, flush=True)
            alive = rng.permutation(np.flatnonzero(pair.ora.alive[:7000]))
            feats = min(feats, len(alive) - dels)
            ops = np.array([(ri.OP_FEAT_UPDATE, w, 0, i) for i, w in enumerate(alive[:feats])] + [(ri.OP_VERTEX_DEL, w, 0, 0) for w in alive[feats:feats + dels]],
                           dtype=np.uint32)
            pair.step(ops, rng.standard_normal((feats, 3)).astype(np.float32))
        pair.check_graph()
        pair.check_aggregates()
    finally:
        pair.close()


@pytest.mark.parametrize("dels,adds", [(1024, 1024), (1, 2048), (3000, 1096), (4096, 1), (9000, 11001)])
def test_long_rows_of_changes_are_put_in_order(dels, adds):
    """Deterministic mode: the changes of one row in two, three, four, five and twenty tiles that are merged. What is appended has to
    be in ascending order, and the terms are sums of it."""
    print("case merged changes", dels, adds, flush=True)
    n, k = 24000, 9500
    rng = np.random.default_rng(dels + adds)
    src = np.arange(1, 1 + k, dtype=np.uint32)
    pair = Pair(n, n + 3, src, np.zeros(k, np.uint32), ri.features(n, 5, 1), ri.make_model("sage_mean", (5, 9, 70, 4), 3), deterministic=True, edge_capacity=40000)
    try:
        gone, new = rng.permutation(src)[:dels], rng.permutation(np.arange(10000, 10000 + adds, dtype=np.uint32))
        ops = np.array([(ri.OP_EDGE_DEL, x, 0, 0) for x in gone] + [(ri.OP_EDGE_ADD, x, 0, 0) for x in new], dtype=np.uint32)
        pair.step(ops[rng.permutation(len(ops))], None)
        pair.check_graph()
        pair.check_aggregates()
        s, d, m = rp.ripple_export_edges(pair.ctx, 1, 40000)
        row = s[:m][d[:m] == 0]
        assert len(row) == k - dels + adds and np.array_equal(row[k - dels:], np.sort(new))
    finally:
        pair.close()


@pytest.mark.parametrize("kind,widths", [("gcn_sum", (70, 9)), ("sage_mean", (12, 300, 24)), ("gcn_wsum", (20, 6)), ("gat", (12, 20, 130)), ("gat", (9, 47))])
def test_a_bootstrap_gives_the_same_bits_again(kind, widths):
    """Destinations whose in-edges lie in several runs of chunks (hubs of up to 9,000) are summed in run order."""
    print("case same bits", kind, widths, flush=True)
    pair, _ = make_pair(n=12000, e=150000, d0=widths[0], kind=kind, widths=widths, seed=81, top_share=0.06, weighted=kind == "gcn_wsum")
    try:
        pair.check_embeddings()
        pair.check_aggregates()
        rows = lambda: [pair.gpu_layer(l) for l in range(1, pair.L + 1)] + [  # noqa: E731
            rp.ripple_get_aggregates(pair.ctx, l, rp.ripple_get_layer_info(pair.ctx, l)[0], n_rows=pair.cap) for l in range(1, pair.L + 1)]
        first = rows()
        for again in range(6):
            rp.ripple_full_infer(pair.ctx)
            for a, b in zip(first, rows()):
                assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    finally:
        pair.close()


@pytest.mark.parametrize("made", [1, 3, 40, 70])
def test_edges_of_vertices_that_a_small_piece_creates(made):
    """Pieces of 9 to 492 operations: edges between a created vertex and a live one, between two created ones, and to a vertex that is
    not alive and stays so (rejected); one creation of a live vertex (rejected)."""
    print("case created endpoints", made, flush=True)
    pair, _ = make_pair(n=900, e=4000, d0=6, kind="sage_mean", widths=(6, 10, 5), seed=91, slack=200)
    rng = np.random.default_rng(92 + made)
    try:
        for turn in range(2):
            first = 900 + 75 * turn
            ops = [(ri.OP_VERTEX_ADD, first + i, 0, i) for i in range(made)] + [(ri.OP_VERTEX_ADD, 7, 0, 0)]
            for i in range(made):
                w = first + i
                ops += [(ri.OP_EDGE_ADD, w, int(x), 0) for x in rng.choice(900, 2, replace=False)] + [(ri.OP_EDGE_ADD, int(x), w, 0) for x in rng.choice(900, 2, replace=False)]
                ops += [(ri.OP_EDGE_ADD, w, first + (i + 1) % made, 0)] if made > 1 else []
                ops += [(ri.OP_EDGE_ADD, w, 1095, 0)]
            ops = np.array(ops, dtype=np.uint32)
            assert len(ops) <= 512
            res, rec, _ = pair.step(ops, rng.standard_normal((made, 6)).astype(np.float32))
            assert res.n_sub_batches == 1 and res.n_rejected == made + 1
        pair.check_graph()
        pair.check_aggregates()
    finally:
        pair.close()
