"""How a hop's in-edges are cut for the wavefronts (rp_run_cut): chunks of 64, 128 and 256 edges, at and next to the numbers of in-edges where
the size changes on a GPU of 256 compute units. Bootstrap and pulled hops, rows of all forms: narrow floats, a lane per column, packed."""
import pytest

import oracle
import paper_2601_12347_amd as rp
from harness import make_pair, make_stream

pytestmark = pytest.mark.gpu

MIX = {"edge_add": 0.35, "edge_del": 0.25, "feat": 0.25, "vadd": 0.08, "vdel": 0.07}
WIDTHS = (20, 72, 130, 47)


@pytest.mark.parametrize("e", [524_288, 524_289, 1_048_577])
@pytest.mark.parametrize("kind,deterministic", [("gcn_sum", False), ("gcn_sum", True), ("gcn_wsum", False), ("gcn_max", False), ("gat", False)])
def test_cuts_of_a_hop(kind, deterministic, e):
    print("case hop cuts", kind, deterministic, e, flush=True)
    pair, graph = make_pair(n=5000, e=e, d0=WIDTHS[0], kind=kind, widths=WIDTHS, seed=421, gamma=2.6, top_share=0.0015, deterministic=deterministic,
                            weighted=kind == "gcn_wsum", edge_capacity=e + 4096)
    try:
        pair.check_embeddings()
        rp.ripple_set_option(pair.ctx, rp.OPT_SCATTER_MODE, 2)
        rp.ripple_set_option(pair.ctx, rp.OPT_SORTED_MESSAGES, 0)
        rp.ripple_set_option(pair.ctx, rp.OPT_SPARSE_FRONTIER, 0)
        stream = make_stream(pair, graph, MIX, 422, weighted=kind == "gcn_wsum")
        for bs in (3, 40):
            ops, payload, _ = stream.next_batch(bs)
            rec = pair.ora.apply_batch(ops, payload)
            res = rp.ripple_apply_updates(pair.ctx, ops, payload)
            assert res.n_applied == int(rec.accepted.sum())
            if kind != "gcn_max":                           # (pruned by value)
                assert list(res.affected[:4]) == [len(s) for s in oracle.affected_sets(pair.ora, rec, pair.model)]
            pair.check_embeddings()
    finally:
        pair.close()
