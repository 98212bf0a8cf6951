"""Row update of attention layers over many rows (k_transform_addend_flat with denominators): remainders of four columns, delta rows,
bf16 rows, and rows that are not finite, each counted once."""
import re

import numpy as np
import pytest

import paper_2601_12347_amd as rp
import ripple_inputs as ri
from harness import Pair

pytestmark = pytest.mark.gpu

N = 70_000                                                 # over the 65,536 rows from which the kernel is taken


def _graph(seed):
    return ri.chung_lu_graph(N, 3 * N, 2.2, 0.004, seed)[:2]


@pytest.mark.parametrize("widths,store", [((8, 47, 6), "f32"), ((8, 67, 5), "f32"), ((8, 64, 5), "f32"), ((12, 13, 4, 1), "f32"), ((8, 46, 7), "bf16")])
def test_rows_of_many_vertices(widths, store):
    print("case attention rows", widths, store, flush=True)
    src, dst = _graph(401)
    model = ri.make_model("gat", widths, 402)
    pair = Pair(N, N + 16, src, dst, ri.features(N, widths[0], 403), model, store=store)
    try:
        pair.check_embeddings()
        ids = np.random.default_rng(404).permutation(N)[:62_000]
        for b in range(2):                                 # the second with the sizes of the first
            ops = np.zeros((len(ids), 4), np.uint32)
            ops[:, 0], ops[:, 1], ops[:, 3] = ri.OP_FEAT_UPDATE, ids, np.arange(len(ids))
            payload = ri.features(len(ids), widths[0], 405 + b)
            pair.ora.apply_batch(ops, payload)
            res = rp.ripple_apply_updates(pair.ctx, ops, payload)
            print(" batch", b, list(res.affected[:pair.L + 1]), flush=True)
            assert min(res.affected[1:pair.L + 1]) >= 65_536
            pair.check_embeddings()
    finally:
        pair.close()


@pytest.mark.parametrize("store", ["f32", "bf16"])
def test_rows_that_are_not_finite_are_counted_once(store):
    """One layer of 47 columns. A row counts if its denominator or a numerator leaves the float range; in 64 bits, rows beyond ten
    times the largest float and rows within a tenth of it are told apart, and the count has to lie between."""
    print("case attention rows out of range", store, flush=True)
    src, dst = _graph(411)
    model = ri.make_model("gat", (8, 47), 412)
    feats = ri.features(N, 8, 413)
    if store == "bf16":                                    # rows are stored rounded: no difference between the two sides' inputs
        feats = (feats.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    lay = model[0]
    lay["att"] = (np.asarray(lay["att"]) * 40.0).astype(np.float32)
    p = feats.astype(np.float64) @ np.asarray(lay["W0"], np.float64)
    att = np.asarray(lay["att"], np.float64)
    s = (p @ att[:47])[src] + (p @ att[47:])[dst]
    e = np.exp(np.where(s > 0, s, 0.2 * s))
    den = np.bincount(dst, e, N)
    num = np.max([np.abs(np.bincount(dst, e * p[src, k], N)) for k in range(47)], axis=0)
    mag = np.maximum(den, num)
    top = float(np.finfo(np.float32).max)
    lo, hi = int((mag > 10 * top).sum()), int((mag > top / 10).sum())
    assert 100 < lo <= hi < 1.3 * lo, (lo, hi)
    ctx = rp.ripple_init_graph(N, N + 16, src, dst, feats, store=store)
    try:
        rp.ripple_load_model(ctx, model)
        with pytest.raises(rp.RippleError) as ei:
            rp.ripple_full_infer(ctx)
        assert ei.value.status == rp.binding.RIPPLE_ERANGE
        n = int(re.search(r"(\d+) row updates", str(ei.value)).group(1))
        print(" rows", lo, n, hi, flush=True)
        assert lo <= n <= hi
    finally:
        rp.ripple_destroy(ctx)
