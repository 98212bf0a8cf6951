"""Reading rows back: pieces through pinned memory, whole tables on the device. Rows are copied, so every number has to be the same."""
import numpy as np
import pytest

import paper_2601_12347_amd as rp

pytestmark = pytest.mark.gpu
PIECE = 65_536                                                # numbers per piece; eight pieces per launch, two launches at a time


def _context(n, d, store):
    rng = np.random.default_rng(n + d)
    rows = rng.standard_normal((n, d), dtype=np.float32)
    src = np.arange(8, dtype=np.uint32)
    ctx = rp.ripple_init_graph(n, n, src, (src + 1) % 8, rows, store=store)
    if store == "bf16":                                       # to nearest even, as the library stores them
        bits = rows.view(np.uint32)
        rows = ((bits + 0x7FFF + ((bits >> 16) & 1)) & np.uint32(0xFFFF0000)).view(np.float32)
    return ctx, rows


@pytest.mark.parametrize("store", ["f32", "bf16"])
@pytest.mark.parametrize("d", [1, 47, 128, 1023])
def test_rows_to_the_host(d, store):
    per = PIECE // d                                          # rows of a piece
    edges = [1, per - 1, per, per + 1, 2 * per + 1, 8 * per, 8 * per + 1, 16 * per + 1, 17 * per - 1]
    n = max(edges) + 5
    ctx, rows = _context(n, d, store)
    try:
        for m in edges:
            print("case reads", d, store, m, flush=True)
            ids = np.random.default_rng(m).permutation(n)[:m].astype(np.uint32)
            got = rp.ripple_get_embeddings(ctx, 0, d, ids=ids)
            assert np.array_equal(got, rows[ids]), f"rows by id, {m}"
            got = rp.ripple_get_embeddings(ctx, 0, d, n_rows=m)
            assert np.array_equal(got, rows[:m]), f"first rows, {m}"
    finally:
        rp.ripple_destroy(ctx)


@pytest.mark.parametrize("n,d", [(1, 1), (3, 1), (1024, 1), (1031, 3), (4096, 5), (5000, 47), (200_003, 47)])
def test_table_on_the_device(n, d):
    import torch
    ctx, rows = _context(max(n, 8), d, "f32")
    try:
        for shift in (0, 1, 2):                               # a caller's array may begin at any multiple of four bytes
            out = torch.full((n * d + 8,), -7.0, device="cuda")
            rp.ripple_get_embeddings(ctx, 0, d, n_rows=n, out=out.data_ptr() + 4 * shift)
            got = out.cpu().numpy()
            assert np.array_equal(got[shift:shift + n * d].reshape(n, d), rows[:n])
            assert (got[:shift] == -7.0).all() and (got[shift + n * d:] == -7.0).all(), "numbers outside the table were written"
    finally:
        rp.ripple_destroy(ctx)


@pytest.mark.parametrize("n_ops", [1, 2, 255, 256, 257, 1500, 30_000])
def test_operations_on_the_device_equal_those_on_the_host(n_ops):
    """The same batch handed over both ways: counts, sets and rows (whole-number features and weights, so sums have no rounding)."""
    import torch
    import ripple_inputs as ri
    n, d = 4000, 8
    rng = np.random.default_rng(n_ops)
    key = rng.permutation(n * n)[:60_000]
    key = key[key // n != key % n]
    src, dst = (key // n).astype(np.uint32), (key % n).astype(np.uint32)
    rows = rng.integers(-3, 4, (n, d)).astype(np.float32)
    model = ri.make_model("gcn_sum", (d, 16, 4), 1)
    for layer in model:
        layer["W0"], layer["b0"] = np.round(layer["W0"] * 4).astype(np.float32), np.zeros_like(layer["b0"])
    cut = src.size - n_ops
    ops = np.zeros((n_ops, 4), np.uint32)
    ops[:, 1], ops[:, 2] = src[cut:], dst[cut:]                # edges that the graph does not have yet
    ops[::3, 0], ops[::3, 1], ops[::3, 2] = 1, src[:ops[::3].shape[0]], dst[:ops[::3].shape[0]]
    results = []
    for on_device in (False, True):
        ctx = rp.ripple_init_graph(n, n, src[:cut], dst[:cut], rows, edge_capacity=2 * src.size)
        try:
            rp.ripple_load_model(ctx, model)
            rp.ripple_full_infer(ctx)
            if on_device:
                held = torch.from_numpy(np.concatenate([np.zeros(1, np.int32), ops.view(np.int32).reshape(-1)])).cuda()
                res = rp.ripple_apply_updates(ctx, held.data_ptr() + 4, None, n_ops=n_ops)
            else:
                res = rp.ripple_apply_updates(ctx, ops, None)
            results.append((res.n_applied, res.n_edges, list(res.affected[:3]), rp.ripple_get_embeddings(ctx, 2, 4, n_rows=n)))
        finally:
            rp.ripple_destroy(ctx)
    assert results[0][:3] == results[1][:3]
    assert np.array_equal(results[0][3], results[1][3])
