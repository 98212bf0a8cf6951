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
