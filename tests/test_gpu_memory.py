"""Device memory that loading a model takes, where a table's size is a choice."""
import numpy as np
import pytest

import paper_2601_12347_amd as rp
import ripple_inputs as ri

pytestmark = pytest.mark.gpu


def _load_bytes(n, d0, kind, widths, edge_capacity):
    """Bytes that ripple_load_model takes on a graph of n vertices without edges."""
    torch = pytest.importorskip("torch")
    torch.zeros(1, device="cuda")
    none = np.zeros(0, np.uint32)
    ctx = rp.ripple_init_graph(n, n, none, none, np.zeros((n, d0), np.float32), edge_capacity=edge_capacity)
    try:
        before = torch.cuda.mem_get_info()[0]
        rp.ripple_load_model(ctx, ri.make_model(kind, widths, 1))
        return before - torch.cuda.mem_get_info()[0]
    finally:
        rp.ripple_destroy(ctx)


def test_lists_of_attention_messages_take_what_they_can_hold():
    """A list holds at most a 64th of the edges' messages: 24 bytes per message, room for a sixteenth of the 84 M entries of the pools (126 MB). What
    else the model takes does not depend on that: segments of long rows (34 MB), parts of cut rows (7 MB)."""
    print("case memory of attention lists", flush=True)
    took = _load_bytes(1000, 8, "gat", (8, 8, 8), 1 << 26)
    print("  MB:", took / 1e6, flush=True)
    assert took <= 200e6


def test_rows_of_narrow_layers_are_not_padded():
    """A layer that is handled project-first keeps three tables of its output's width per vertex (H, the aggregate, what has been sent): 16 columns take
    42 numbers per vertex more than 2 do."""
    print("case memory of narrow rows", flush=True)
    n = 2_000_000
    took = {d: _load_bytes(n, 32, "gcn_sum", (32, d), 1000) for d in (2, 16)}
    print("  MB:", {d: b / 1e6 for d, b in took.items()}, flush=True)
    assert took[16] - took[2] >= 0.95 * 42 * 4 * n
