"""The workloads this library's speed is judged by: what a user has it do, through the public entry points.

A case is an evolving graph with a model on it. One pass of an "update" case is what a trigger-based inference service
does per batch: ripple_apply_updates, then the vertices whose prediction the batch could change and their new rows. One
pass of a "bootstrap" case is ripple_full_infer and the whole prediction table.

A context keeps its state from batch to batch, so a case holds a ring of batches: some forward ones, then their
inverses in reverse order (edges taken out again or put back, features restored, created vertices deleted and deleted
ones created again with their edges). Every pass applies the next one, the graph never drifts away from its size, and
no batch meets the graph that it met a moment ago.
"""
import functools
import json
import math

import numpy as np
import torch

import paper_2601_12347_amd as rp
import ripple_inputs as ri
from ripple_inputs.graphs import (OP_EDGE_ADD, OP_EDGE_DEL, OP_FEAT_UPDATE, OP_VERTEX_ADD, OP_VERTEX_DEL, PowerLaw)

# The graphs of ripple_inputs.CONFIGS, and one between the sparse and the dense one.
TINY = dict(n=2_000, e=20_000, gamma=2.1, top=0.015)
SPARSE = dict(n=169_343, e=1_166_243, gamma=2.1, top=0.01)
MID = dict(n=612_257, e=30_929_573, gamma=2.3, top=0.0008)
DENSE = dict(n=2_449_029, e=123_718_280, gamma=2.3, top=0.0002)

# run: "update" or "bootstrap". bs: updates per batch; of them `vops` are vertex creations (8 edges each) and as many
# deletions, the rest 50 % new edges, 30 % deleted edges, 20 % feature rows. given: where the batch lies. read: what is read back after it:
# the affected predictions as host arrays, as device tensors, or the whole table on the device.
BASE = dict(run="update", kind="sage_mean", d0=128, hidden=256, classes=40, layers=3, store="f32", bs=1000, vops=0.0, given="host", read="device",
            deterministic=False)


def _case(name, graph, **kw):
    return dict(BASE, name=name, **graph, **kw)


def listed():
    return [
        # the smallest graph and an ordinary batch for it: launches and host work
        _case("tiny_gcn_sum_b100", TINY, kind="gcn_sum", d0=32, hidden=64, classes=16, layers=2, bs=100, read="host"),
        # one update at a time, the answer wanted at once on the host: latency
        _case("sparse_sage_mean_b1", SPARSE, bs=1, read="host"),
        # the everyday batch on a citation-sized graph
        _case("sparse_sage_mean_b100", SPARSE, bs=100),
        # a large batch on it, four layers, bit-reproducible sums (audited results)
        _case("sparse_sage_det_b1000", SPARSE, layers=4, bs=1000, deterministic=True),
        # vertices come and go; two-stage (MLP) updates
        _case("sparse_gin_vertex_ops_b1000", SPARSE, kind="gin_sum", bs=1000, vops=0.05),
        # monotonic aggregation; the whole table is read (the affected set is pruned by value)
        _case("sparse_gcn_max_b1000", SPARSE, kind="gcn_max", bs=1000, read="all"),
        # attention on a graph between the two large ones
        _case("mid_gat_b300", MID, kind="gat", d0=100, classes=47, bs=300),
        # edge weights, widths that are multiples of nothing
        _case("mid_wsum_odd_b1777", MID, kind="gcn_wsum", d0=75, hidden=190, classes=23, bs=1777),
        # the bootstrap: every vertex, every layer
        _case("mid_bootstrap", MID, run="bootstrap", d0=100, classes=47, read="all", bs=0),
        # a small batch on the large graph: everything that scans the graph shows
        _case("dense_sage_mean_b100", DENSE, d0=100, classes=47, bs=100),
        # the headline workload, batches handed over on the device
        _case("dense_sage_mean_b10000", DENSE, d0=100, classes=47, bs=10_000, given="device"),
        # bf16 rows, no self term, vertices come and go
        _case("dense_gcn_sum_bf16_b10000", DENSE, kind="gcn_sum", d0=100, classes=47, store="bf16", bs=10_000, vops=0.01, given="device"),
    ]


def _between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sage_mean", "sage_mean", "sage_mean", "gcn_sum", "gin_sum", "gcn_wsum", "gcn_max", "gat"])
    run = "bootstrap" if rng.random() < 0.1 else "update"
    n = _between(rng, 2_000, 2_449_029)
    # what reads whole in-rows again (max, attention, the bootstrap) stays below the largest listed case's cost on the middle graph
    if kind in ("gcn_max", "gat") or run == "bootstrap":
        n = _between(rng, 2_000, 612_257)
    if kind == "gin_sum":                          # two products per row
        n = min(n, 1_000_000)
    e = int(n * math.exp(rng.uniform(math.log(6.9), math.log(50.5))))
    bs = _between(rng, 1, min(10_000, max(100, n // 100)))
    if kind in ("gcn_max", "gat"):
        bs = min(bs, 1000)
        e = min(e, 8_000_000 if kind == "gcn_max" else 30_929_573)
    c = dict(BASE, run=run, kind=kind, n=n, e=e, gamma=rng.choice([2.1, 2.2, 2.3]), top=min(0.015, 400.0 / n + 0.0002),
             d0=rng.choice([32, 100, 128, rng.randint(17, 160)]), hidden=rng.choice([64, 128, 256, 256, 256, rng.randint(33, 256)]),
             classes=rng.choice([16, 40, 47, rng.randint(2, 64)]), layers=rng.choice([2, 3, 3]), bs=bs if run == "update" else 0,
             given=rng.choice(["host", "device"]), read="all" if run == "bootstrap" or kind == "gcn_max" else "device")
    if kind in ("gcn_sum", "sage_mean") and rng.random() < 0.25:
        c["store"] = "bf16"
    if run == "update" and c["read"] == "device" and bs <= 100 and n <= 200_000:
        c["read"] = "host"
    if run == "update" and rng.random() < 0.3:
        c["vops"] = rng.choice([0.01, 0.05])
    if kind in ("sage_mean", "gin_sum", "gcn_sum") and n <= 200_000 and rng.random() < 0.15:
        c["deterministic"] = True
    return c


# ---- inputs ----------------------------------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _sampler(n, gamma, top, seed, dev):
    """Vertices of a Chung-Lu degree law (ripple_inputs.PowerLaw), drawn on the device."""
    law = PowerLaw(n, gamma, top, seed)
    perm = torch.from_numpy(law.perm).to(dev)

    def pick(k, gen):
        u = torch.rand(k, generator=gen, device=dev, dtype=torch.float64)
        x = (u * (law.hi - law.lo) + law.lo).pow_(1.0 / law.e).sub_(law.i0).floor_()
        return perm[x.clamp_(0, n - 1).long()]

    return pick


def _edges(pick_out, pick_in, n, count, gen, taken=None):
    """`count` distinct edges u * n + v without loops, sorted; none of those in `taken` (sorted)."""
    keys = torch.empty(0, dtype=torch.int64, device=gen.device)
    while keys.numel() < count:
        k = int((count - keys.numel()) * 1.1) + 256
        u, v = pick_out(k, gen), pick_in(k, gen)
        new = (u * n + v)[u != v]
        if taken is not None:
            at = torch.searchsorted(taken, new).clamp_(max=taken.numel() - 1)
            new = new[taken[at] != new]
        keys = torch.unique(torch.cat([keys, new]))
    if keys.numel() > count:
        keep = torch.ones(keys.numel(), dtype=torch.bool, device=gen.device)
        keep[torch.randperm(keys.numel(), generator=gen, device=gen.device)[: keys.numel() - count]] = False
        keys = keys[keep]
    return keys


def _inputs(case, seed):
    """Graph, features, weights and the forward batches, as device tensors (vertex ids int64)."""
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(1_000_003 * seed + 17)
    n, bs = case["n"], case["bs"]
    pick_out, pick_in = _sampler(n, case["gamma"], case["top"], 7 * seed + 1, dev), _sampler(n, case["gamma"], case["top"], 7 * seed + 2, dev)
    g = {"keys": _edges(pick_out, pick_in, n, case["e"], gen), "H0": torch.randn(n, case["d0"], generator=gen, device=dev)}
    if case["kind"] == "gcn_wsum":
        g["w"] = torch.rand(case["e"], generator=gen, device=dev) * 1.5 + 0.25
    if case["run"] == "bootstrap":
        return g
    # K batches; the kinds of all their updates in one pool, so that single-update batches take turns
    k = 10 if bs < 10 else 4
    total = k * bs
    n_v = int(round(case["vops"] * total))
    rest = total - 2 * n_v
    n_add, n_del = int(round(0.5 * rest)), int(round(0.3 * rest))
    n_feat = min(rest - n_add - n_del, n // 4)
    n_add = rest - n_del - n_feat
    rng = np.random.default_rng(seed + 5)
    who = rng.permutation(n)                       # deleted vertices first, then those whose features are replaced
    gone = np.sort(who[:n_v])
    feat = who[n_v:n_v + n_feat]
    gone_d = torch.zeros(n, dtype=torch.bool, device=dev)
    if n_v:
        gone_d[torch.from_numpy(gone).to(dev)] = True
    touches = lambda keys: gone_d[keys // n] | gone_d[keys % n]  # noqa: E731
    add = _edges(pick_out, pick_in, n, n_add + 64 + n_add // 4, gen, taken=g["keys"])
    add = add[~touches(add)]
    add = add[torch.randperm(add.numel(), generator=gen, device=dev)[:n_add]].cpu().numpy()
    old = torch.unique(torch.randint(0, case["e"], (2 * n_del + 64,), generator=gen, device=dev))
    old = old[~touches(g["keys"][old])]
    old = old[torch.randperm(old.numel(), generator=gen, device=dev)[:n_del]]
    cut = g["keys"][old].cpu().numpy()
    g["cut_w"] = g["w"][old].cpu().numpy() if "w" in g else np.zeros(len(cut), np.float32)
    incident = np.zeros(0, np.int64)
    incident_w = np.zeros(0, np.float32)
    if n_v:
        sel = torch.nonzero(touches(g["keys"])).reshape(-1)
        incident = g["keys"][sel].cpu().numpy()
        if "w" in g:
            incident_w = g["w"][sel].cpu().numpy()
    alive = np.ones(n, bool)
    alive[gone] = False
    peers = np.flatnonzero(alive)
    kinds = np.repeat([0, 1, 2, 3, 4], [len(add), len(cut), n_feat, n_v, n_v])
    rng.shuffle(kinds)
    kinds = np.array_split(kinds, k)
    g["batches"] = []
    at = [0] * 5
    feat_d = torch.from_numpy(feat).to(dev)
    old_rows = g["H0"][feat_d].cpu().numpy() if n_feat else np.zeros((0, case["d0"]), np.float32)
    gone_rows = g["H0"][torch.from_numpy(gone).to(dev)].cpu().numpy() if n_v else np.zeros((0, case["d0"]), np.float32)
    left = np.ones(len(incident), bool)            # edges of deleted vertices that still exist
    order = rng.permutation(len(gone))
    for kk in kinds:
        c = np.bincount(kk, minlength=5)
        part = [slice(at[j], at[j] + c[j]) for j in range(5)]
        at = [a + int(x) for a, x in zip(at, c)]
        b = {"add": add[part[0]], "add_w": rng.uniform(0.25, 1.75, int(c[0])).astype(np.float32), "cut": cut[part[1]], "cut_w": g["cut_w"][part[1]],
             "feat": feat[part[2]], "feat_old": old_rows[part[2]], "feat_new": rng.standard_normal((int(c[2]), case["d0"]), dtype=np.float32)}
        ids = np.arange(n + part[3].start, n + part[3].stop)          # created vertices, eight edges each
        near = peers[np.argsort(rng.random((len(ids), 64)), axis=1)[:, :8] * (len(peers) // 64) + rng.integers(0, len(peers) // 64, (len(ids), 8))] \
            if len(ids) else np.zeros((0, 8), np.int64)
        out = rng.random((len(ids), 8)) < 0.5
        own = np.broadcast_to(ids[:, None], near.shape)
        b["new"], b["new_rows"] = ids, rng.standard_normal((len(ids), case["d0"]), dtype=np.float32)
        b["new_u"], b["new_v"] = np.where(out, own, near), np.where(out, near, own)
        b["new_w"] = rng.uniform(0.25, 1.75, near.shape).astype(np.float32)
        w = order[part[4]]
        b["gone"], b["gone_rows"] = gone[w], gone_rows[w]
        if n_v:
            mine = left & (np.isin(incident // n, b["gone"]) | np.isin(incident % n, b["gone"]))
            left &= ~mine
            b["gone_edges"], b["gone_w"] = incident[mine], incident_w[mine] if "w" in g else np.zeros(int(mine.sum()), np.float32)
        else:
            b["gone_edges"], b["gone_w"] = np.zeros(0, np.int64), np.zeros(0, np.float32)
        g["batches"].append(b)
    return g


def _ops(kind, u, v=None, row=None):
    o = np.zeros((len(u), 4), np.uint32)
    o[:, 0], o[:, 1] = kind, u
    if v is not None:
        o[:, 2] = v
    if row is not None:
        o[:, 3] = row
    return o


def _encode(b, n, back, weighted, rng):
    """One batch as operation records and its feature rows, forwards or backwards."""
    bits = lambda w: w.view(np.uint32) if weighted else None  # noqa: E731
    if not back:
        rows = np.concatenate([b["feat_new"], b["new_rows"]])
        loose = np.concatenate([_ops(OP_EDGE_ADD, b["add"] // n, b["add"] % n, bits(b["add_w"])), _ops(OP_EDGE_DEL, b["cut"] // n, b["cut"] % n),
                                _ops(OP_FEAT_UPDATE, b["feat"], None, np.arange(len(b["feat"]))), _ops(OP_VERTEX_DEL, b["gone"])])
        new = np.stack([np.concatenate([_ops(OP_VERTEX_ADD, b["new"][i:i + 1], None, [len(b["feat"]) + i]),
                                        _ops(OP_EDGE_ADD, b["new_u"][i], b["new_v"][i], bits(b["new_w"][i]))])
                        for i in range(len(b["new"]))]).reshape(-1, 4) if len(b["new"]) else np.zeros((0, 4), np.uint32)
        return np.ascontiguousarray(np.concatenate([new, loose[rng.permutation(len(loose))]])), rows
    rows = np.concatenate([b["feat_old"], b["gone_rows"]])
    loose = np.concatenate([_ops(OP_EDGE_DEL, b["add"] // n, b["add"] % n), _ops(OP_EDGE_ADD, b["cut"] // n, b["cut"] % n, bits(b["cut_w"])),
                            _ops(OP_FEAT_UPDATE, b["feat"], None, np.arange(len(b["feat"]))), _ops(OP_VERTEX_DEL, b["new"])])
    again = np.concatenate([_ops(OP_VERTEX_ADD, b["gone"], None, len(b["feat"]) + np.arange(len(b["gone"]))),
                            _ops(OP_EDGE_ADD, b["gone_edges"] // n, b["gone_edges"] % n, bits(b["gone_w"]))])
    return np.ascontiguousarray(np.concatenate([again, loose[rng.permutation(len(loose))]])), rows


class _Service:
    """A context and the ring of batches that comes in."""

    def __init__(self, case, seed):
        self.case, self.ctx, self.turn = case, None, 0
        g = _inputs(case, seed)
        n, dev = case["n"], _device()
        self.widths = (case["d0"],) + (case["hidden"],) * (case["layers"] - 1) + (case["classes"],)
        self.cap = n + max(128, int(4 * case["bs"] * case["vops"]) + 128)
        src, dst = ((k.to(torch.int32).cpu().numpy().view(np.uint32)) for k in (g["keys"] // n, g["keys"] % n))
        H0 = g["H0"].cpu().numpy()
        kw = dict(store=case["store"], edge_capacity=int(case["e"] * 1.05) + 65536)
        if "w" in g:
            self.ctx = rp.ripple_init_graph_weighted(n, self.cap, src, dst, g["w"].cpu().numpy(), H0, **kw)
        else:
            self.ctx = rp.ripple_init_graph(n, self.cap, src, dst, H0, **kw)
        if case["deterministic"]:
            rp.ripple_set_option(self.ctx, rp.OPT_DETERMINISTIC, 1)
        rp.ripple_load_model(self.ctx, ri.make_model(case["kind"], self.widths, seed + 3))
        rp.ripple_full_infer(self.ctx)
        self.ring = []
        if case["run"] == "update":
            rng = np.random.default_rng(seed + 6)
            both = [(b, False) for b in g["batches"]] + [(b, True) for b in reversed(g["batches"])]
            for b, back in both:
                ops, rows = _encode(b, n, back, "w" in g, rng)
                if case["given"] == "device":
                    ops, rows = torch.from_numpy(ops.view(np.int32)).to(dev), torch.from_numpy(rows).to(dev)
                self.ring.append((ops, rows))
        # where the caller wants the answer: the set and its predictions (room for every vertex), or the whole table
        if case["read"] == "all":
            self.rows = torch.zeros(n, case["classes"], device=dev)
        elif case["read"] == "device":
            self.ids, self.size = torch.zeros(self.cap, dtype=torch.int32, device=dev), torch.zeros(1, dtype=torch.int32, device=dev)
            self.rows = torch.zeros(self.cap, case["classes"], device=dev)
        else:
            self.ids, self.rows = np.zeros(self.cap, np.uint32), np.zeros((self.cap, case["classes"]), np.float32)

    def __del__(self):
        if self.ctx is not None:
            rp.ripple_destroy(self.ctx)
            self.ctx = None


def prepare(case, seed):
    return _Service(case, seed)


def run(s):
    c, ctx = s.case, s.ctx
    L, d = c["layers"], c["classes"]
    out = {}
    if c["run"] == "bootstrap":
        rp.ripple_full_infer(ctx)
    else:
        ops, rows = s.ring[s.turn % len(s.ring)]
        s.turn += 1
        if c["given"] == "device":
            res = rp.ripple_apply_updates(ctx, ops.data_ptr(), rows.data_ptr() if len(rows) else None, n_ops=len(ops), n_feat_rows=len(rows))
        else:
            res = rp.ripple_apply_updates(ctx, ops, rows)
        out["edges"], out["applied"] = res.n_edges, res.n_applied
        if c["read"] != "all":
            out["affected"] = list(res.affected[:L + 1])
    out["rows"] = s.rows
    if c["read"] == "all":
        rp.ripple_get_embeddings(ctx, L, d, n_rows=c["n"], out=s.rows.data_ptr())
        return out
    out["ids"] = s.ids
    n = res.affected[L]
    if c["read"] == "host":
        ids, _ = rp.ripple_get_affected(ctx, L, n)
        s.ids[:n] = ids
        rp.ripple_get_embeddings(ctx, L, d, ids=ids, out=s.rows[:n])
        return out
    out["size"] = s.size
    rp.ripple_get_affected_static(ctx, L, s.ids.data_ptr(), s.cap, s.size.data_ptr())
    rp.ripple_get_embeddings(ctx, L, d, ids=s.ids.data_ptr(), n_rows=n, out=s.rows.data_ptr())
    return out


# ---- what a pass cannot do without -----------------------------------------------------------------------------
@functools.lru_cache(maxsize=64)
def _hops(text):
    """Mean over the forward batches: vertices per hop, messages per hop, their distinct destinations."""
    case = json.loads(text)
    n, dev = case["n"], _device()
    g = _inputs(case, 1)
    src, dst = g["keys"] // n, g["keys"] % n
    self_term = case["kind"].startswith(("sage", "gin")) or case["kind"] == "gat"
    L = case["layers"]
    a, m, t = np.zeros(L + 1), np.zeros(L + 1), np.zeros(L + 1)
    for b in g["batches"]:
        mark = lambda ids: torch.zeros(n, dtype=torch.bool, device=dev).index_fill_(0, torch.from_numpy(np.unique(ids[ids < n])).to(dev), True)  # noqa: E731
        sinks = mark(np.concatenate([b["add"] % n, b["cut"] % n, b["new_v"].reshape(-1), b["gone_edges"] % n]))
        front = mark(b["feat"])
        a[0] += len(b["feat"]) + len(b["new"])
        for l in range(1, L + 1):
            go = front[src]
            hit = torch.zeros(n, dtype=torch.bool, device=dev)
            hit[dst[go]] = True
            m[l] += int(go.sum())
            t[l] += int(hit.sum())
            front = (hit | sinks | front) if self_term else (hit | sinks)
            a[l] += int(front.sum()) + len(b["new"])
    k = len(g["batches"])
    return (a / k).tolist(), (m / k).tolist(), (t / k).tolist()


def work(case):
    """Per hop: an index per message, each sender's row once, each destination's sum read and written, each refreshed row
    written, the products of the refreshed rows; then the rows that are read back."""
    s = 2 if case["store"] == "bf16" else 4
    widths = [case["d0"]] + [case["hidden"]] * (case["layers"] - 1) + [case["classes"]]
    nbytes = flops = 0.0
    if case["run"] == "bootstrap":
        N = case["n"]
        a, m, t = [N] * len(widths), [case["e"]] * len(widths), [N] * len(widths)
    else:
        a, m, t = _hops(json.dumps({k: v for k, v in case.items() if k != "name"}, sort_keys=True))
        nbytes += 16 * case["bs"] + 2 * 4 * a[0] * case["d0"]
    for l in range(1, len(widths)):
        d_in, d_out = widths[l - 1], widths[l]
        w = min(d_in, d_out)                       # a sum may travel before or after the linear map
        nbytes += 4 * m[l] + a[l - 1] * w * s + (1 if case["run"] == "bootstrap" else 2) * t[l] * w * 4 + a[l] * d_out * s
        flops += m[l] * w
        if case["kind"].startswith("gin"):
            flops += 2 * a[l] * (d_in * case["hidden"] + case["hidden"] * d_out)
        else:
            flops += 2 * a[l] * d_in * d_out + (2 * a[l - 1] * d_in * d_out if case["kind"].startswith("sage") else 0)
    read = case["n"] if case["read"] == "all" else a[-1]
    nbytes += read * case["classes"] * (s + 4) + (4 * read if case["read"] != "all" else 0)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # 32-bit sums in another order, over up to four layers; bf16 rows: one rounding step of the stored rows
    return {"rel": 1e-2, "max": 0.2} if case["store"] == "bf16" else {"rel": 2e-5, "max": 2e-3}
