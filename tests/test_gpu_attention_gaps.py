"""A listed attention hop in which few vertices are recomputed and hundreds of thousands are patched: the recomputed ones lie far apart in the hop's list,
with patched ones in between. The batch must not take longer than twice what it takes with the scan of all in-rows that the list replaces."""
import time

import numpy as np
import pytest

import paper_2601_12347_amd as rp
import ripple_inputs as ri

pytestmark = pytest.mark.gpu


def _star(n, spread):
    """0 -> 1 and 0 -> `spread` vertices at equal distances; 1 -> all the others: a new row of 0 makes 0, 1 and those `spread` vertices be recomputed
    at hop 2, from one in-edge each, and the others be patched. (The last vertex is one of the `spread`.)"""
    apart = n - 1 - np.arange(spread) * ((n - 2) // spread)
    others = np.setdiff1d(np.arange(2, n), apart)
    src = np.concatenate([np.zeros(1 + spread, np.int64), np.ones(len(others), np.int64)])
    dst = np.concatenate([[1], apart, others])
    return src.astype(np.uint32), dst.astype(np.uint32)


def _context(n, src, dst, widths, sorted_messages, edge_capacity):
    ctx = rp.ripple_init_graph(n, n, src, dst, ri.features(n, widths[0], 3), edge_capacity=edge_capacity)
    rp.ripple_load_model(ctx, ri.make_model("gat", widths, 4))
    rp.ripple_full_infer(ctx)
    rp.ripple_set_option(ctx, rp.OPT_SORTED_MESSAGES, sorted_messages)
    rp.ripple_set_option(ctx, rp.OPT_SPARSE_FRONTIER, 0)
    return ctx


# 2^20 walked edges and more are listed in larger tiles
@pytest.mark.parametrize("n,spread", [(400_000, 1), (400_000, 1000), (1_200_000, 3)])
def test_few_recomputed_vertices_far_apart(n, spread):
    print("case attention gaps", n, spread, flush=True)
    widths = (8, 8, 8)
    src, dst = _star(n, spread)
    times, rows = {}, {}
    for mode in (2, 0):
        ctx = _context(n, src, dst, widths, mode, 40_000_000)
        try:
            rng, best = np.random.default_rng(5), np.inf
            for b in range(6):
                row = rng.standard_normal((1, widths[0])).astype(np.float32)
                t0 = time.perf_counter()
                res = rp.ripple_apply_updates(ctx, np.array([(ri.OP_FEAT_UPDATE, 0, 0, 0)], np.uint32), row)
                best = min(best, time.perf_counter() - t0)
                assert list(res.affected[:3]) == [1, 2 + spread, n] and res.hop_mode[2] == (4 if mode else 0)
            times[mode], rows[mode] = best, rp.ripple_get_embeddings(ctx, 2, widths[2], n_rows=n)
        finally:
            rp.ripple_destroy(ctx)
    print("  ms, listed / scanned:", [round(1e3 * times[m], 3) for m in (2, 0)], flush=True)
    # six patches of three roundings each, of terms up to 1 / GAT_CANCEL = 1,000 times what is left of them: 6 * 3 * 2^-24 * 1,000
    assert np.abs(rows[2] - rows[0]).max() <= 1.1e-3 * np.abs(rows[0]).max()
    assert times[2] <= 2.0 * times[0]
