"""Products of many rows (k_split_stream: fp32 numbers as three bf16 parts on the bf16 matrix cores) at small sizes, forced with
RIPPLE_OPT_STREAM_TRANSFORM = 2, against the oracle and against the other kernels' products (option 0); and the tiles of
k_transform_split, forced with RIPPLE_OPT_SPLIT_MFMA."""
import numpy as np
import pytest

import oracle
import paper_2601_12347_amd as rp
import ripple_inputs as ri
from harness import Pair, make_pair, make_stream
from ripple_inputs.graphs import OP_FEAT_UPDATE

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.4, "edge_del": 0.25, "feat": 0.2, "vadd": 0.08, "vdel": 0.07}

# widths on both sides of every multiple the kernel works in (4 numbers, 16 and 32 k, 32 and 64 columns), one and two slices of k,
# 64, 128 and 256 padded columns, odd row strides; every kind of row (aggregate, own row, GIN sum, hidden row) and both stores
SHAPES = [("sage_mean", (75, 190, 190, 23), "f32", False), ("gcn_wsum", (75, 190, 190, 23), "f32", True), ("gin_sum", (33, 256, 200, 129), "f32", False),
          ("sage_mean", (129, 65, 128, 40), "f32", False), ("gcn_sum", (17, 100, 70), "f32", False), ("gat", (100, 256, 129, 47), "f32", False),
          ("gcn_max", (31, 255, 97), "f32", False), ("sage_mean", (100, 256, 256, 47), "bf16", False), ("gcn_sum", (66, 250, 33), "bf16", False),
          ("gcn_sum", (100, 256, 100), "bf16", False), ("gcn_sum", (65, 201, 33), "bf16", False), ("sage_mean", (33, 129, 47), "bf16", False)]


@pytest.mark.parametrize("kind,widths,store,weighted", SHAPES)
def test_products_of_every_shape(kind, widths, store, weighted):
    print("case products", kind, widths, store, flush=True)
    pair, graph = make_pair(n=700, e=7000, d0=widths[0], kind=kind, widths=widths, seed=271, slack=64, weighted=weighted, store=store)
    rp.ripple_set_option(pair.ctx, rp.OPT_STREAM_TRANSFORM, 2)
    rp.ripple_full_infer(pair.ctx)
    stream = make_stream(pair, graph, MIX, 273, weighted=weighted)
    try:
        pair.check_embeddings()
        for b, bs in enumerate([1, 40, 200]):
            print(" batch", b, bs, flush=True)
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
            pair.check_aggregates()
    finally:
        pair.close()


def _rows(kind, widths, feats, option):
    n, e = 400, 3000
    src, dst, _, _ = ri.chung_lu_graph(n, e, 2.1, 0.03, 281)
    model = ri.make_model(kind, widths, 283)
    ctx = rp.ripple_init_graph(n, n, src, dst, feats)
    rp.ripple_load_model(ctx, model)
    try:
        rp.ripple_set_option(ctx, rp.OPT_STREAM_TRANSFORM, option)
        rp.ripple_full_infer(ctx)
        return [rp.ripple_get_embeddings(ctx, l, widths[l], n_rows=n) for l in range(1, len(widths))]
    finally:
        rp.ripple_destroy(ctx)


@pytest.mark.parametrize("kind", ["sage_mean", "gcn_sum", "gin_sum"])
def test_numbers_that_have_no_parts(kind):
    """Infinities, NaNs and numbers that bf16 rounds to infinity: the same elements are infinite (with the same sign), NaN and finite as
    with fp32 products, and the finite ones agree. One layer without activation: 256 sums of at most 50 rows keep 1e-5 of the largest."""
    widths = (100, 200)
    feats = ri.features(400, 100, 282)
    feats[3, 5], feats[40, 99], feats[77, 0], feats[200, 31], feats[310, 64] = np.inf, -np.inf, np.nan, 3.4e38, -3.395e38
    on, off = _rows(kind, widths, feats, 2)[0], _rows(kind, widths, feats, 0)[0]
    assert np.array_equal(np.isnan(on), np.isnan(off)) and np.array_equal(np.isposinf(on), np.isposinf(off)) and np.array_equal(np.isneginf(on), np.isneginf(off))
    assert np.isnan(on).any() and (np.abs(on[np.isfinite(on)]) > 1e36).any()
    assert np.isinf(on).any() or kind == "gin_sum"          # (a second product makes NaNs of them)
    fin = np.isfinite(on)
    scale = np.maximum(np.where(fin, np.abs(off), 0).max(axis=1, keepdims=True), 1e-30)
    assert (np.abs(np.where(fin, on, 0) - np.where(fin, off, 0)) / scale).max() <= 1e-5


@pytest.mark.parametrize("scale", [1e-30, 1e-10, 1.0, 1e10, 1e30])
def test_rows_of_any_magnitude(scale):
    """The parts of a number are relative to it: rows of 1e-30 and of 1e30 are as exact as rows of 1 (weights of about 0.1, biases 0)."""
    widths = (100, 200)
    feats = (ri.features(400, 100, 284) * np.float32(scale)).astype(np.float32)
    n = 400
    src, dst, _, _ = ri.chung_lu_graph(n, 3000, 2.1, 0.03, 281)
    model = ri.make_model("sage_mean", widths, 285)
    for layer in model:
        layer["b0"] = np.zeros_like(layer["b0"])
    errs = {}
    for option in (2, 0):
        pair = Pair(n, n, src, dst, feats, model)
        try:
            rp.ripple_set_option(pair.ctx, rp.OPT_STREAM_TRANSFORM, option)
            rp.ripple_full_infer(pair.ctx)
            want = oracle.full_recompute(pair.ora, model)[1]
            got = rp.ripple_get_embeddings(pair.ctx, 1, widths[1], n_rows=n).astype(np.float64)
            errs[option] = np.linalg.norm((got - want) / scale) / np.linalg.norm(want / scale)
        finally:
            pair.close()
    print("scale %g: error against 64 bits %.2e, fp32 products %.2e" % (scale, errs[2], errs[0]), flush=True)
    assert errs[2] <= max(1.1 * errs[0], 1.5e-7)


# rows of [own | aggregate] (2 d_in of k, from a layer that concatenates and keeps no self term), of more than 256 k, and matrices of
# 64, 128, 256 and 512 padded columns; project-first layers take the same matrix with its first d_in rows alone
@pytest.mark.parametrize("kind,widths,self_cache,project_first", [
    ("sage_mean", (100, 132, 260, 47), False, True), ("sage_mean", (100, 132, 260, 47), False, False), ("sage_mean", (200, 260, 64, 130), False, False),
    ("sage_mean", (75, 129, 31), False, False), ("gcn_sum", (300, 270, 40), True, False), ("gin_sum", (260, 300, 129), True, True)])
def test_split_products_of_wide_rows(kind, widths, self_cache, project_first):
    print("case wide rows", kind, widths, self_cache, project_first, flush=True)
    pair, graph = make_pair(n=500, e=4000, d0=widths[0], kind=kind, widths=widths, seed=291, slack=64, self_cache=self_cache,
                            project_first=project_first, split=True)
    stream = make_stream(pair, graph, MIX, 293)
    try:
        pair.check_embeddings()
        for b, bs in enumerate([1, 40, 200]):
            print(" batch", b, bs, flush=True)
            ops, payload, _ = stream.next_batch(bs)
            pair.step(ops, payload)
            pair.check_aggregates()
    finally:
        pair.close()


@pytest.mark.parametrize("rows,weights", [(1e-33, 1.0), (1e-36, 1.0), (1.0, 1e-33), (1.0, 1e-36), (1e-20, 1e-16), (1e20, 1e-13)])
@pytest.mark.parametrize("way", ["stream", "tiles"])
def test_parts_of_tiny_numbers(way, rows, weights):
    """Rows or weights near the smallest normal number: their parts keep all bits, in both kernels that split. Bound as for rows of any magnitude
    (sums of 1e-37 are themselves rounded at 1e-45, 1e-8 of them)."""
    widths, n = (100, 200), 400
    feats = (ri.features(n, 100, 284) * np.float32(rows)).astype(np.float32)
    src, dst, _, _ = ri.chung_lu_graph(n, 3000, 2.1, 0.03, 281)
    model = ri.make_model("sage_mean", widths, 285)
    for layer in model:
        layer["b0"] = np.zeros_like(layer["b0"])
        layer["W0"] = (layer["W0"] * np.float32(weights)).astype(np.float32)
    errs = {}
    for kernel in (way, "fp32"):
        pair = Pair(n, n, src, dst, feats, model, split=kernel == "tiles")
        try:
            rp.ripple_set_option(pair.ctx, rp.OPT_STREAM_TRANSFORM, 2 if kernel == "stream" else 0)
            rp.ripple_full_infer(pair.ctx)
            want = oracle.full_recompute(pair.ora, model)[1]
            got = rp.ripple_get_embeddings(pair.ctx, 1, widths[1], n_rows=n).astype(np.float64)
            scale = np.abs(want).max()
            errs[kernel] = np.linalg.norm((got - want) / scale) / np.linalg.norm(want / scale)
        finally:
            pair.close()
    print("rows %g weights %g %s: error against 64 bits %.2e, fp32 products %.2e" % (rows, weights, way, errs[way], errs["fp32"]), flush=True)
    assert errs[way] <= max(1.1 * errs["fp32"], 1.5e-7)


def _two_batches(kind, widths, store, self_cache, split, stream):
    """Every layer after the bootstrap on a table with special numbers, after a batch that brings more of them and after one that replaces all
    of them by ordinary ones. No activations: a NaN stays one."""
    n = 400
    src, dst, _, _ = ri.chung_lu_graph(n, 3000, 2.1, 0.03, 281)
    feats = ri.features(n, widths[0], 282)
    feats[3, 5], feats[40, -1], feats[77, 0], feats[200, 31], feats[310, 64] = np.inf, -np.inf, np.nan, 1e35, -2e35
    model = ri.make_model(kind, widths, 283)
    for layer in model:
        layer["act_inner"] = layer["act_out"] = "none"
    ctx = rp.ripple_init_graph(n, n, src, dst, feats, store=store)
    try:
        for option, value in ((rp.OPT_SELF_CACHE, int(self_cache)), (rp.OPT_SPLIT_MFMA, split), (rp.OPT_STREAM_TRANSFORM, stream), (rp.OPT_BF16_MFMA, 0),
                              (rp.OPT_SPARSE_FRONTIER, 0)):
            rp.ripple_set_option(ctx, option, value)
        rp.ripple_load_model(ctx, model)
        rp.ripple_full_infer(ctx)
        rows = lambda: [rp.ripple_get_embeddings(ctx, l, widths[l], n_rows=n) for l in range(1, len(widths))]
        out = [rows()]
        odd, even = [3, 40, 77, 200, 310, 11, 12, 13], ri.features(8, widths[0], 286)
        special = even.copy()
        special[5, 7], special[6, 40], special[7, 2] = -np.inf, np.nan, 3e35
        for vs, payload in (([11, 12, 13], special[5:]), (odd, even)):
            ops = np.array([(OP_FEAT_UPDATE, v, 0, i) for i, v in enumerate(vs)], np.uint32)
            rp.ripple_apply_updates(ctx, ops, np.ascontiguousarray(payload))
            out.append(rows())
        return out
    finally:
        rp.ripple_destroy(ctx)


def _bootstrap_pattern(kind, widths):
    n = 400
    src, dst, _, _ = ri.chung_lu_graph(n, 3000, 2.1, 0.03, 281)
    feats = ri.features(n, widths[0], 282)
    feats[3, 5], feats[40, -1], feats[77, 0], feats[200, 31], feats[310, 64] = np.inf, -np.inf, np.nan, 1e35, -2e35
    model = ri.make_model(kind, widths, 283)
    for layer in model:
        layer["act_inner"] = layer["act_out"] = "none"
    with np.errstate(all="ignore"):
        return [np.isfinite(h) for h in oracle.full_recompute(oracle.GraphState(n, n, src, dst, feats), model)[1:]]


# kinds of rows: aggregate; own row, and aggregate with a cached row; [own | aggregate]; GIN sum and hidden row; project-first with one and two
# products. (100, 200, 72) has 256 and 128 padded columns, (128, 60, 40) 64
@pytest.mark.parametrize("store", ["f32", "bf16"])
@pytest.mark.parametrize("kind,widths,self_cache", [("gcn_sum", (100, 200, 72), True), ("sage_mean", (100, 200, 72), True), ("sage_mean", (100, 200, 72), False),
                                                    ("gin_sum", (100, 200, 72), True), ("gcn_sum", (128, 60, 40), True), ("sage_mean", (128, 60, 40), True)])
def test_sums_that_are_not_finite_are_made_again(kind, widths, self_cache, store):
    """Through the tiles and the streaming kernel: the same elements are infinite (with the same sign), NaN and finite as with fp32 products, in the layer that
    meets the numbers and in the one that receives its rows of changes. Finite elements agree to 1e-5 of their row's largest (bf16 rows: a
    rounding of 2^-8, amplified by a layer of sums) until differences of numbers of 1e35 remain."""
    print("case not finite", kind, widths, self_cache, store, flush=True)
    want = _two_batches(kind, widths, store, self_cache, 0, 0)
    assert np.isnan(want[0][0]).any() and np.isnan(want[2][1]).any()
    if kind == "gin_sum":                                   # (its first product has no fp32 kernel: the bootstrap's pattern is the oracle's)
        exact = _bootstrap_pattern(kind, widths)
        assert all(np.array_equal(np.isfinite(a), b) for a, b in zip(want[0], exact))
    for way, split, stream in (("tiles", 1, 0), ("stream", 0, 2)):
        got = _two_batches(kind, widths, store, self_cache, split, stream)
        for step in range(3):
            for l in range(len(widths) - 1):
                a, b = got[step][l], want[step][l]
                where = (way, step, l + 1)
                assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isposinf(a), np.isposinf(b)) and np.array_equal(np.isneginf(a), np.isneginf(b)), where
                if step < 2:
                    fin = np.isfinite(b)
                    x, y = np.where(fin, a, 0).astype(np.float64), np.where(fin, b, 0).astype(np.float64)
                    err = (np.abs(x - y) / np.maximum(np.abs(y).max(axis=1, keepdims=True), 1e-30)).max()
                    assert err <= (1e-5 if store == "f32" else 2.0 ** -5), where
