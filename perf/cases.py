"""Timed cases of the library: what a program does with it, through the
binding's public entry points, over the range of sizes that the tests, the
benchmarks and the workload presets of this repository use.

Every case is a dict of plain values.  ``kind`` says which calls a pass makes:

  run       gsp_run on a loaded graph, then its membership and modularity
  learned   the same with the shipped pruning network in front of the scans
  leiden    the same with GSP-Leiden's refinement in every pass
  batch     gsp_run_batch on loaded graphs, then memberships and modularities
  load_run  a new graph in host memory: load, run, membership, modularity
  evaluate  modularity and disconnected communities of a given membership
  train     one epoch of the pruning network's training

``graph`` names the input law (seeded here, drawn on the GPU): ``sbm``
(planted partition), ``rmat``, ``dcsbm`` (degree-corrected, power-law degrees
and community sizes) and ``road`` (a lattice subdivided into chains), with
the parameters of the presets in ``gsp_inputs``.  ``weights`` is ``unit``,
``f32`` or ``f64``.
"""
import math
import os
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2402_11454_amd as gsp

_DEV = "cuda:0"


def listed():
    return [
        # the smallest graph of the batch law: pure latency, every level tiny
        {"name": "run-sbm-1k", "kind": "run", "graph": "sbm", "n": 1013, "degree": 12.0, "mixing": 0.3,
         "weights": "unit"},
        # the 10,000-vertex planted partition, the first workload of the presets
        {"name": "run-sbm-10k", "kind": "run", "graph": "sbm", "n": 10000, "degree": 20.0, "mixing": 0.2,
         "weights": "unit"},
        # a program that meets one new graph after another: load from host
        # memory, run once, fetch the result
        {"name": "load-run-sbm-100k", "kind": "load_run", "graph": "sbm", "n": 100003, "degree": 20.0, "mixing": 0.3,
         "weights": "f32"},
        # web-like graph, unit weights, loaded order (below the degree-order size)
        {"name": "run-rmat-20", "kind": "run", "graph": "rmat", "scale": 20, "edge_factor": 16, "weights": "unit"},
        # the largest: web-like, fp32 weights, stored in degree order
        {"name": "run-rmat-24", "kind": "run", "graph": "rmat", "scale": 24, "edge_factor": 16, "weights": "f32"},
        # social-network-like graph at the full size of its preset
        {"name": "run-dcsbm-4m", "kind": "run", "graph": "dcsbm", "n": 4000000, "mixing": 0.3, "weights": "f32"},
        # learned pruning (the gate's inference and its history)
        {"name": "learned-dcsbm-1m", "kind": "learned", "graph": "dcsbm", "n": 1000001, "mixing": 0.3,
         "weights": "f32", "threshold": 0.1},
        # GSP-Leiden on a web-like graph with weights
        {"name": "leiden-rmat-20", "kind": "leiden", "graph": "rmat", "scale": 20, "edge_factor": 16,
         "weights": "f32"},
        # road / k-mer class: average degree about 2, long chains, many levels
        {"name": "run-road-15m", "kind": "run", "graph": "road", "side": 1500, "weights": "unit"},
        # many uneven graphs at once
        {"name": "batch-64", "kind": "batch", "graph": "sbm", "graphs": 64, "n_max": 200000, "weights": "unit"},
        # quality check of a membership from elsewhere
        {"name": "evaluate-rmat-22", "kind": "evaluate", "graph": "rmat", "scale": 22, "edge_factor": 16,
         "weights": "f32"},
        # training of the pruning network on recorded rows, mini-batches of
        # the recipe's size (forward, backward, Adam)
        {"name": "train-512k", "kind": "train", "rows": 524288, "batch": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "learned", "leiden", "batch", "load_run", "evaluate", "train"])
    if kind == "train":
        return {"kind": kind, "rows": _log_int(rng, 8192, 2000000), "batch": rng.choice([1024, 2048, 4096, 8192])}
    if kind == "batch":
        return {"kind": kind, "graph": "sbm", "graphs": _log_int(rng, 4, 64), "n_max": _log_int(rng, 4000, 200000),
                "weights": rng.choice(["unit", "f32"])}
    weights = rng.choice(["unit", "f32", "f32", "f64"])
    if kind == "load_run":
        return {"kind": kind, "graph": "sbm", "n": _log_int(rng, 1000, 1000000), "degree": rng.uniform(4.0, 40.0),
                "mixing": rng.uniform(0.1, 0.5), "weights": weights}
    graph = rng.choice(["sbm", "rmat", "rmat", "dcsbm", "dcsbm", "road"] if kind == "run" else ["sbm", "rmat", "dcsbm"])
    case = {"kind": kind, "graph": graph, "weights": weights}
    if graph == "sbm":
        case.update(n=_log_int(rng, 1000, 1000000), degree=rng.uniform(4.0, 40.0), mixing=rng.uniform(0.1, 0.5))
    elif graph == "rmat":
        case.update(scale=rng.randint(14, 22), edge_factor=rng.randint(4, 20))
    elif graph == "dcsbm":
        case.update(n=_log_int(rng, 10000, 4000000), mixing=rng.uniform(0.1, 0.5))
    else:
        case.update(side=_log_int(rng, 100, 1500), weights="unit")
    if kind == "learned":
        case["threshold"] = 0.7 if graph == "rmat" else 0.1
    return case


# ------------------------------------------------------------------ inputs

_RANGE = {"sbm": (1.0, 4.0), "dcsbm": (1.0, 4.0), "rmat": (1.0, 10.0), "road": (1.0, 4.0)}


def _gen(seed):
    g = torch.Generator(device=_DEV)
    g.manual_seed(int(seed))
    return g


def _rand(m, g):
    return torch.rand(m, generator=g, device=_DEV, dtype=torch.float64)


def _pair_weights(key, n, lo, hi, seed, dtype):
    """A weight per unordered pair: a mix of the pair and the seed, so that
    both directions of an edge get the same value."""
    u, v = key // n, key % n
    h = torch.minimum(u, v) * n + torch.maximum(u, v) + (seed * 0x1F123BB5 + 1) % (1 << 61)
    h = (h ^ ((h >> 31) & 0x1FFFFFFFF)) * 0x3F58476D1CE4E5B9
    h = (h ^ ((h >> 29) & 0x7FFFFFFFF)) * 0x14D049BB133111EB
    x = ((h >> 20) & 0xFFFFFF).to(torch.float32) * 2.0 ** -24
    return (lo + (hi - lo) * x).to(dtype)


def _csr(u, v, n, weights, law, seed):
    """Symmetric CSR on the GPU of the undirected pairs (u, v): self-loops
    dropped, duplicates removed, rows sorted."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.cat([u * n + v, v * n + u])
    del u, v, keep
    key = torch.sort(key)[0]
    if key.numel():
        first = torch.ones(key.numel(), dtype=torch.bool, device=_DEV)
        first[1:] = key[1:] != key[:-1]
        key = key[first]
        del first
    off = torch.searchsorted(key, torch.arange(n + 1, device=_DEV, dtype=torch.int64) * n)
    w = None
    if weights != "unit":
        lo, hi = _RANGE[law]
        w = _pair_weights(key, n, lo, hi, seed, torch.float32 if weights == "f32" else torch.float64)
    col = (key % n).to(torch.int32)
    return off, col, w


def _relabel(n, g):
    return torch.randperm(n, generator=g, device=_DEV)


def _sbm_pairs(n, degree, mixing, g):
    blocks = max(1, int(round(n / 100)))
    m_in, m_out = int(n * degree * (1.0 - mixing) / 2), int(n * degree * mixing / 2)
    u = torch.randint(n, (m_in,), generator=g, device=_DEV)
    b = u * blocks // n
    lo, hi = (b * n + blocks - 1) // blocks, ((b + 1) * n + blocks - 1) // blocks
    v = lo + (_rand(m_in, g) * (hi - lo)).long()
    uo = torch.randint(n, (m_out,), generator=g, device=_DEV)
    vo = torch.randint(n, (m_out,), generator=g, device=_DEV)
    p = _relabel(n, g)
    return p[torch.cat([u, uo])], p[torch.cat([v, vo])]


def _rmat_pairs(scale, edge_factor, g):
    n, m = 1 << scale, edge_factor << scale
    u = torch.zeros(m, dtype=torch.int64, device=_DEV)
    v = torch.zeros(m, dtype=torch.int64, device=_DEV)
    for _ in range(scale):
        r = torch.rand(m, generator=g, device=_DEV)
        u.mul_(2).add_((r >= 0.76).long())
        v.mul_(2).add_((((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).long())
    p = _relabel(n, g)
    return p[u], p[v]


def _power_law(m, alpha, lo, hi, g):
    """m draws of a truncated power law x^-alpha on [lo, hi]."""
    a, b, e = float(lo) ** (1 - alpha), float(hi + 1) ** (1 - alpha), 1.0 / (1 - alpha)
    return (a + (b - a) * _rand(m, g)).pow(e).long().clamp(lo, hi)


def _dcsbm_pairs(n, mixing, g):
    k = _power_law(n, 2.5, 5, min(5000, max(50, n // 20)), g)
    size = _power_law(max(16, n // 20), 1.5, 20, min(50000, max(100, n // 10)), g)
    end = torch.cumsum(size, 0)
    # vertices stand in random order, so consecutive runs are communities
    comm = torch.searchsorted(end, torch.arange(n, device=_DEV), right=True).clamp(max=size.numel() - 1)
    frac = k.double() * (1.0 - mixing)
    k_in = (frac + _rand(n, g)).long()
    stub = torch.repeat_interleave(torch.arange(n, device=_DEV), k_in)
    sc = comm[stub]
    cnt = torch.bincount(sc, minlength=size.numel())
    start = torch.cumsum(cnt, 0) - cnt
    u, c = stub[::2], sc[::2]
    v = stub[start[c] + (_rand(u.numel(), g) * cnt[c]).long()]
    out = torch.repeat_interleave(torch.arange(n, device=_DEV), k - k_in)
    uo = out[::2]
    vo = out[torch.randint(max(out.numel(), 1), (uo.numel(),), generator=g, device=_DEV)]
    p = _relabel(n, g)
    return p[torch.cat([u, uo])], p[torch.cat([v, vo])]


def _road_pairs(side, g):
    at = torch.arange(side * side, device=_DEV).view(side, side)
    a = torch.cat([at[:, :-1].reshape(-1), at[:-1, :].reshape(-1)])
    b = torch.cat([at[:, 1:].reshape(-1), at[1:, :].reshape(-1)])
    keep = _relabel(a.numel(), g)[:int(0.7 * a.numel())]
    a, b = a[keep], b[keep]
    inner = _relabel(a.numel(), g) % 9
    base = side * side + torch.cumsum(inner, 0) - inner
    n = side * side + int(inner.sum())
    e = torch.repeat_interleave(torch.arange(a.numel(), device=_DEV), inner + 1)
    first = torch.cumsum(inner + 1, 0) - (inner + 1)
    t = torch.arange(e.numel(), device=_DEV) - first[e]
    u = torch.where(t == 0, a[e], base[e] + t - 1)
    v = torch.where(t == inner[e], b[e], base[e] + t)
    p = _relabel(n, g)
    return p[u], p[v], n


def _graph(case, seed):
    """(n, offsets, cols, weights or None) of the case's graph, on the GPU."""
    g = _gen(seed)
    law = case["graph"]
    if law == "sbm":
        n = case["n"]
        u, v = _sbm_pairs(n, case["degree"], case["mixing"], g)
    elif law == "rmat":
        n = 1 << case["scale"]
        u, v = _rmat_pairs(case["scale"], case["edge_factor"], g)
    elif law == "dcsbm":
        n = case["n"]
        u, v = _dcsbm_pairs(n, case["mixing"], g)
    else:
        u, v, n = _road_pairs(case["side"], g)
    off, col, w = _csr(u, v, n, case["weights"], law, seed)
    return n, off, col, w


def _batch(case, seed):
    g = _gen(seed)
    r = random.Random(case["graphs"])   # the sizes belong to the case, the graphs to the seed
    got = []
    for k in range(case["graphs"]):
        n = int(round(math.exp(r.uniform(math.log(1e3), math.log(case["n_max"])))))
        u, v = _sbm_pairs(n, r.uniform(4.0, 40.0), r.uniform(0.1, 0.5), g)
        off, col, w = _csr(u, v, n, case["weights"], "sbm", seed + k)
        got.append(SimpleNamespace(n=n, offsets=off.cpu().numpy(), cols=col.cpu().numpy(),
                                   weights=None if w is None else w.cpu().numpy()))
    return got


def _net():
    return np.fromfile(os.path.join(os.path.dirname(gsp.__file__), "pruner_dcsbm.f32"), dtype="<f4")


def _train_rows(case, seed):
    """Feature rows in the gate's ranges and labels of a noisy rule on them,
    a third of them positive, and He-uniform starting parameters."""
    g = _gen(seed)
    rows = case["rows"]
    x = torch.rand(rows, 8, generator=g, device=_DEV)
    x[:, 6] = torch.randint(3, (rows,), generator=g, device=_DEV).float() * 0.5
    x[:, 2] = 2.0 * x[:, 2] - 1.0
    z = 1.5 * x[:, 7] + x[:, 2] - 0.8 * x[:, 1] + 0.5 * (x[:, 6] - 0.5) - 0.9
    y = (z + 0.5 * torch.randn(rows, generator=g, device=_DEV) > 0).to(torch.uint8)
    r = np.random.default_rng(seed)
    p = np.zeros(gsp.GATE_PARAMS, np.float32)
    p[0:512] = r.uniform(-1, 1, 512) * math.sqrt(6 / 8)
    p[576:4672] = r.uniform(-1, 1, 4096) * math.sqrt(6 / 64)
    p[4736:4800] = r.uniform(-1, 1, 64) * math.sqrt(6 / 64)
    return x.contiguous(), y.contiguous(), p


def _labels(n, seed):
    """A membership from elsewhere: communities of power-law sizes over
    vertices in random order."""
    g = _gen(seed + 1)
    size = _power_law(max(16, n // 20), 1.5, 20, max(100, n // 100), g)
    comm = torch.searchsorted(torch.cumsum(size, 0), torch.arange(n, device=_DEV), right=True)
    return comm[_relabel(n, g)].clamp(max=n - 1).to(torch.int32)


def prepare(case, seed):
    kind = case["kind"]
    ctx = gsp.Context(0)
    state = {"kind": kind, "ctx": ctx, "opt": gsp.default_options()}
    if kind == "train":
        state["x"], state["y"], state["params"] = _train_rows(case, seed)
        state["batch"] = case["batch"]
        torch.cuda.synchronize()
        return state
    if kind == "batch":
        ctx.load_batch(_batch(case, seed))
        state["graphs"] = case["graphs"]
        return state
    n, off, col, w = _graph(case, seed)
    if kind == "load_run":
        state["csr"] = tuple(None if t is None else t.cpu().numpy() for t in (off, col, w))
        return state
    torch.cuda.synchronize()
    ctx.load(off, col, w)
    del off, col, w
    torch.cuda.empty_cache()
    if kind == "learned":
        ctx.pruner_set(_net())
        state["opt"] = gsp.default_options(prune_mode=gsp.PRUNE_LEARNED, prune_threshold=case["threshold"])
    elif kind == "leiden":
        state["opt"] = gsp.default_options(leiden=1)
    elif kind == "evaluate":
        state["membership"] = _labels(n, seed)
        torch.cuda.synchronize()
    state["out"] = torch.empty(n, dtype=torch.int32, device=_DEV)
    return state


def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "train":
        params, loss = ctx.pruner_train(state["params"], state["x"], state["y"], batch=state["batch"], epochs=1,
                                        lr=2e-3, pos_weight=2.0)
        return {"params": params, "loss": loss.astype(np.float32)}
    if kind == "batch":
        ctx.run_batch(1e-2, 10, options=state["opt"])
        return {"membership": np.concatenate([ctx.batch_membership(k) for k in range(state["graphs"])]),
                "modularity": ctx.batch_modularity()}
    if kind == "evaluate":
        return {"modularity": ctx.modularity(state["membership"]),
                "disconnected": ctx.count_disconnected(state["membership"])}
    if kind == "load_run":
        ctx.load(*state["csr"])
        ctx.run(1e-2, 10, options=state["opt"])
        return {"membership": ctx.membership(), "modularity": ctx.result_modularity()}
    ctx.run(1e-2, 10, options=state["opt"])
    return {"membership": ctx.membership(state["out"]), "modularity": ctx.result_modularity()}


# -------------------------------------------------------------------- work

def _size(case):
    """(vertices, directed entries) of the case's graphs, about."""
    if case["graph"] == "sbm" and case["kind"] == "batch":
        mean = (case["n_max"] - 1e3) / math.log(case["n_max"] / 1e3)
        return case["graphs"] * mean, case["graphs"] * mean * 22.0
    if case["graph"] == "sbm":
        return case["n"], case["n"] * case["degree"]
    if case["graph"] == "rmat":
        return 1 << case["scale"], 2.0 * (case["edge_factor"] << case["scale"])
    if case["graph"] == "dcsbm":
        return case["n"], case["n"] * 13.5
    return 6.6 * case["side"] ** 2, 14.0 * case["side"] ** 2


def work(case):
    """Graph read once, membership written once (evaluate: read); training:
    every row read once, forward and backward of the 8-64-64-1 network."""
    if case["kind"] == "train":
        return {"bytes": case["rows"] * 33.0, "flops": case["rows"] * 6.0 * (8 * 64 + 64 * 64 + 64)}
    n, nnz = _size(case)
    wb = {"unit": 0, "f32": 4, "f64": 8}[case["weights"]]
    return {"bytes": nnz * (4.0 + wb) + n * 12.0, "flops": 2.0 * nnz}


# ------------------------------------------------------------------- exact

def _exact_modularity(case, seed):
    n, off, col, w = _graph(case, seed)
    m = _labels(n, seed).long()
    deg = off[1:] - off[:-1]
    row = torch.repeat_interleave(torch.arange(n, device=_DEV), deg)
    w = torch.ones(col.numel(), dtype=torch.float64, device=_DEV) if w is None else w.double()
    m2 = w.sum()
    inside = w[m[row] == m[col.long()]].sum()
    total = torch.zeros(n, dtype=torch.float64, device=_DEV).index_add_(0, m[row], w)
    return float(inside / m2 - ((total / m2) ** 2).sum())


def _exact_train(case, seed):
    """The epoch in 64 bits: mean pos-weighted cross-entropy, Adam (0.9,
    0.999, 1e-8)."""
    x, y, p0 = _train_rows(case, seed)
    x, y = x.double(), y.double()
    p = torch.from_numpy(p0).double().to(_DEV)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    lr, pw, batch, losses = float(np.float32(2e-3)), 2.0, case["batch"], []
    for t, lo in enumerate(range(0, x.shape[0], batch), 1):
        xb, yb = x[lo:lo + batch], y[lo:lo + batch]
        w1, b1 = p[0:512].view(64, 8), p[512:576]
        w2, b2 = p[576:4672].view(64, 64), p[4672:4736]
        w3, b3 = p[4736:4800], p[4800]
        h1 = torch.relu(xb @ w1.t() + b1)
        h2 = torch.relu(h1 @ w2.t() + b2)
        z = h2 @ w3 + b3
        sp = torch.nn.functional.softplus
        losses.append((pw * yb * sp(-z) + (1 - yb) * sp(z)).mean())
        dz = (-pw * yb * torch.sigmoid(-z) + (1 - yb) * torch.sigmoid(z)) / xb.shape[0]
        d2 = dz[:, None] * w3[None, :] * (h2 > 0)
        d1 = (d2 @ w2) * (h1 > 0)
        g = torch.cat([(d1.t() @ xb).reshape(-1), d1.sum(0), (d2.t() @ h1).reshape(-1), d2.sum(0), h2.t() @ dz,
                       dz.sum().reshape(1)])
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - lr * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return p.cpu().numpy(), np.array([float(torch.stack(losses).mean())], dtype=np.float64)


def exact(case, seed):
    """Modularity of a given membership and the trained parameters in 64
    bits; a run's own partition has no closed form."""
    if case["kind"] == "evaluate":
        return {"modularity": _exact_modularity(case, seed), "disconnected": None}
    if case["kind"] == "train" and case["rows"] // case["batch"] <= 2000:
        params, loss = _exact_train(case, seed)
        return {"params": params, "loss": loss}
    return None
