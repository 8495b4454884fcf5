"""Performance cases: the work that programs have this library do, through
its public entry points (``paper_2008_05718_amd.binding``).

A case is a dict of plain values.  ``kind`` "bc": one ``Graph.run`` over a list
of sources and one ``Graph.scores`` into a device tensor, on a handle made
beforehand (a program keeps the handle and runs source lists on it).  ``kind``
"policy_grad": one loss and gradient of the level-policy network.  Graphs are
drawn on the GPU from the seed alone: R-MAT (social and web graphs), damaged
grids (road networks), uniform random graphs, and unions of many
preferential-attachment graphs, in the sizes of ``workloads.py`` and of the
tests.
"""
from __future__ import annotations

import math
import os
from types import SimpleNamespace

import numpy as np
import torch

import paper_2008_05718_amd
from paper_2008_05718_amd import binding as b

_POLICY = os.path.join(os.path.dirname(paper_2008_05718_amd.__file__), "policy_weights.npy")


def listed():
    return [
        # the smallest call: one source of a small graph, where launches and host work count
        {"name": "rmat10_one_source", "kind": "bc", "family": "rmat", "scale": 10, "ef": 8, "sources": 1},
        # all sources of one small graph (ER of 2000 vertices, mean degree 8)
        {"name": "er2000_all", "kind": "bc", "family": "er", "n": 2000, "deg": 8.0, "sources": 0},
        # one batch of sources on a mid-sized graph: a sample for an estimate
        {"name": "rmat14_64", "kind": "bc", "family": "rmat", "scale": 14, "ef": 16, "sources": 64},
        # a few sources, one at a time: the per-source engine
        {"name": "rmat18_per_source", "kind": "bc", "family": "rmat", "scale": 18, "ef": 16, "sources": 32,
         "batch": 1},
        # the ordinary power-law run
        {"name": "rmat18_2048", "kind": "bc", "family": "rmat", "scale": 18, "ef": 16, "sources": 2048},
        # the largest graph of the benchmark, learned level policy, a slice of its sources
        {"name": "rmat22_1024_learned", "kind": "bc", "family": "rmat", "scale": 22, "ef": 16, "sources": 1024,
         "learned": True},
        # road-like: many thin levels, path counts beyond 64 bits (FP64 mode)
        {"name": "grid1024_256", "kind": "bc", "family": "grid", "L": 1024, "shortcuts": 0.001, "sources": 256},
        # directed web graph, ragged number of sources
        {"name": "rmat18_directed_1000", "kind": "bc", "family": "rmat", "scale": 18, "ef": 16, "sources": 1000,
         "directed": True},
        # integer arc weights: shortest paths by relaxation
        {"name": "rmat16_weighted_512", "kind": "bc", "family": "rmat", "scale": 16, "ef": 16, "sources": 512,
         "weights": 100},
        # many small graphs of uneven size in one handle, every 8th vertex a source
        {"name": "union96_small", "kind": "bc", "family": "union", "graphs": 96, "lo": 1000, "hi": 16000, "every": 8},
        # many graphs up to 1e5 vertices, every 64th vertex a source
        {"name": "union64_large", "kind": "bc", "family": "union", "graphs": 64, "lo": 1000, "hi": 100000,
         "every": 64},
        # one full-batch training step's loss and gradient of the policy network
        {"name": "policy_grad_4096", "kind": "policy_grad", "samples": 4096},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    what = rng.choice(["rmat", "rmat", "rmat", "directed", "weighted", "weighted", "grid", "grid", "er", "union",
                       "per_source", "policy_grad"])
    if what == "policy_grad":
        return {"kind": "policy_grad", "samples": int(_log(rng, 100, 16384))}
    c = {"kind": "bc"}
    if what == "er":
        c.update(family="er", n=int(_log(rng, 200, 4000)), deg=round(rng.uniform(4.0, 16.0), 2), sources=0)
    elif what == "grid":
        L = int(_log(rng, 48, 1024))
        # without shortcuts the number of levels grows with L: small ones only
        sc = rng.choice([0.001, 0.01]) if L > 128 else rng.choice([0.0, 0.001])
        c.update(family="grid", L=L, shortcuts=sc, sources=int(_log(rng, 1, 256)))
    elif what == "union":
        c.update(family="union", graphs=rng.randint(8, 64), lo=500, hi=int(_log(rng, 4000, 60000)),
                 every=rng.choice([16, 64]))
    elif what == "per_source":
        c.update(family="rmat", scale=rng.randint(10, 18), ef=16, sources=rng.randint(1, 32), batch=1)
    elif what == "weighted":
        c.update(family="rmat", scale=rng.randint(10, 16), ef=rng.choice([8, 16]),
                 sources=int(_log(rng, 1, 512)), weights=rng.choice([4, 100, 1000]),
                 directed=rng.random() < 0.3)
    else:
        scale = rng.randint(10, 20)
        c.update(family="rmat", scale=scale, ef=rng.choice([8, 16]), sources=int(_log(rng, 2, 2048)))
        if what == "directed":
            c["directed"] = True
        elif rng.random() < 0.3:
            c["learned"] = True
    if c.get("sources") and c["family"] == "rmat":
        c["sources"] = min(c["sources"], 1 << (c["scale"] - 2))
    return c


# ------------------------------------------------------------------- graphs
def _csr(n, u, v, directed=False):
    """int32 CSR on the GPU: self-loops and duplicates dropped, rows ascending."""
    keep = u != v
    u, v = u[keep], v[keep]
    keys = u * n + v
    if not directed:
        keys = torch.cat([keys, v * n + u])
    keys = torch.unique(keys)
    rows = keys // n
    rp = torch.zeros(n + 1, dtype=torch.int64, device=keys.device)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rp.to(torch.int32), (keys - rows * n).to(torch.int32)


def _rmat(case, g):
    scale, n = case["scale"], 1 << case["scale"]
    E = case["ef"] * n
    u = torch.zeros(E, dtype=torch.int64, device="cuda")
    v = torch.zeros_like(u)
    for bit in range(scale):
        r = torch.rand(E, device="cuda", generator=g)
        u |= (r >= 0.76).to(torch.int64) << bit
        v |= (((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).to(torch.int64) << bit
    perm = torch.randperm(n, device="cuda", generator=g)
    return n, perm[u], perm[v]


def _grid(case, g):
    L = case["L"]
    ids = torch.arange(L * L, device="cuda").view(L, L)
    u = torch.cat([ids[:, :-1].reshape(-1), ids[:-1, :].reshape(-1)])
    v = torch.cat([ids[:, 1:].reshape(-1), ids[1:, :].reshape(-1)])
    keep = torch.rand(u.numel(), device="cuda", generator=g) >= 0.10
    u, v = u[keep], v[keep]
    k = int(round(case["shortcuts"] * u.numel()))
    s = torch.randint(0, L * L, (2, k), device="cuda", generator=g)
    return L * L, torch.cat([u, s[0]]), torch.cat([v, s[1]])


def _er(case, g):
    n = case["n"]
    e = torch.randint(0, n, (2, int(n * case["deg"] / 2)), device="cuda", generator=g)
    return n, e[0], e[1]


def _union(case, seed, g):
    """Preferential attachment: every vertex sends 4 edges to endpoints drawn
    from the edges before it (an endpoint that is itself such a draw is
    followed back until a vertex is known)."""
    # sizes spread evenly over the logarithm, in an order of the seed's
    k = np.random.default_rng(seed).permutation(case["graphs"])
    sizes = case["lo"] * (case["hi"] / case["lo"]) ** ((k + 0.5) / case["graphs"])
    off = np.concatenate([[0], np.cumsum(sizes.astype(np.int64))])
    n = int(off[-1])
    toff = torch.from_numpy(off).cuda()
    gi = torch.repeat_interleave(torch.arange(case["graphs"], device="cuda"), toff[1:] - toff[:-1])
    base = toff[gi]  # first vertex of each vertex's graph
    slot = torch.arange(4 * n, device="cuda")
    src = slot // 4
    first = 4 * base[src]  # first edge slot of the graph
    r = ((2 * (slot - first) + 1) * torch.rand(4 * n, device="cuda", generator=g, dtype=torch.float64)).to(torch.int64)
    at, odd = first + r // 2, (r & 1).bool()  # the edge drawn, and whether its far end is meant
    for _ in range(64):
        more = odd & odd[at] & (at < slot)
        if not bool(more.any()):
            break
        at = torch.where(more, at[at], at)
    dst = torch.where(odd, src[at[at]], src[at])
    return n, src, dst, off.astype(np.int32)


def _weights(n, rp, col, case, seed):
    """One weight in [1, weights] per edge (both arcs carry it), or per arc of
    a directed graph."""
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), (rp[1:] - rp[:-1]).to(torch.int64))
    c = col.to(torch.int64)
    key = row * n + c if case.get("directed") else torch.minimum(row, c) * n + torch.maximum(row, c)
    x = (key + seed * 7919) * 0x9E3779B1 & 0x7FFFFFFFFFFF
    x = ((x >> 15) ^ x) * 0x85EBCA6B & 0x7FFFFFFFFFFF
    return (1 + ((x >> 13) ^ x) % case["weights"]).to(torch.int32)


def _inputs(case, seed):
    """Graph (device CSR, weights or None, vertex offsets or None) and host sources."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    off = None
    if case["family"] == "union":
        n, u, v, off = _union(case, seed, g)
    else:
        n, u, v = {"rmat": _rmat, "grid": _grid, "er": _er}[case["family"]](case, g)
    rp, col = _csr(n, u, v, bool(case.get("directed")))
    wt = _weights(n, rp, col, case, seed) if case.get("weights") else None
    if off is not None:
        srcs = np.concatenate([np.arange(off[i], off[i + 1], case["every"]) for i in range(len(off) - 1)])
    elif case["sources"]:
        pool = torch.nonzero(rp[1:] > rp[:-1]).view(-1)
        srcs = pool[torch.randperm(pool.numel(), device="cuda", generator=g)[:case["sources"]]].cpu().numpy()
    else:
        srcs = np.arange(n)
    return rp, col, wt, off, srcs.astype(np.int32)


def _grad_inputs(case, seed):
    """Weights near a trained net's, features in [0, 1] and log2 microseconds,
    three of the nine outputs measured per sample (as collected samples have it)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = case["samples"]
    w = torch.randn(b.BC_MLP_PARAMS, device="cuda", generator=g) * 0.2
    X = torch.rand(n, b.BC_MLP_IN, device="cuda", generator=g)
    Y = torch.rand(n, b.BC_MLP_OUT, device="cuda", generator=g) * 8 + 2
    pick = torch.randint(0, 3, (n, 1), device="cuda", generator=g)
    mask = (torch.arange(b.BC_MLP_OUT, device="cuda") // 3 == pick).to(torch.uint8)
    return w, X, Y, mask


# -------------------------------------------------------------------- passes
def prepare(case, seed):
    if case["kind"] == "policy_grad":
        return {"in": _grad_inputs(case, seed), "loss": torch.zeros(1, device="cuda"),
                "grad": torch.zeros(b.BC_MLP_PARAMS, device="cuda")}
    rp, col, wt, off, srcs = _inputs(case, seed)
    G = b.Graph(SimpleNamespace(row_ptr=rp, col_idx=col, weights=wt, vtx_offsets=off,
                                directed=bool(case.get("directed"))))
    if case.get("learned"):
        G.load_policy(np.load(_POLICY))
    return {"graph": G, "srcs": srcs, "opts": {"batch": case.get("batch", 0)},
            "out": torch.zeros(G.n, dtype=torch.float64, device="cuda")}


def run(state):
    stream = torch.cuda.current_stream()
    if "graph" not in state:
        w, X, Y, mask = state["in"]
        b.bc_mlp_loss_grad_noalloc(w, X, Y, mask, state["loss"], state["grad"], stream=stream)
        return {"loss": state["loss"], "grad": state["grad"]}
    state["graph"].run(state["srcs"], stream=stream, **state["opts"])
    return state["graph"].scores(state["out"], stream=stream)


def _sizes(case):
    """(vertices, stored arcs, sources) to expect."""
    if case["family"] == "rmat":
        n = 1 << case["scale"]
        arcs = case["ef"] * n * (0.93 if case.get("directed") else 1.82)
    elif case["family"] == "grid":
        n = case["L"] ** 2
        arcs = 3.6 * n
    elif case["family"] == "er":
        n = case["n"]
        arcs = n * case["deg"]
    else:
        n = case["graphs"] * (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
        arcs = 8 * n
    s = case["sources"] if case.get("sources") else n / case.get("every", 1)
    return n, arcs, s


def work(case):
    """The graph, the sources and the scores once; per (arc, source) one
    addition forward and a multiplication and an addition backward (for a
    union, of the source's own graph)."""
    if case["kind"] == "policy_grad":
        n, p = case["samples"], b.BC_MLP_PARAMS
        return {"bytes": n * (b.BC_MLP_IN * 4 + b.BC_MLP_OUT * 5) + 8 * p + 4, "flops": 6 * n * p}
    n, arcs, s = _sizes(case)
    own = arcs
    if case["family"] == "union":  # mean of size^2 over mean of size, log-uniform sizes
        own = 8 * (case["lo"] + case["hi"]) / 2
    return {"bytes": 4 * n + arcs * (8 if case.get("weights") else 4) + 4 * s + 8 * n, "flops": 3 * own * s}


# ----------------------------------------------------- the same in 64 bits
def _sparse(rp, col):
    n = rp.numel() - 1
    return torch.sparse_csr_tensor(rp, col, torch.ones(col.numel(), dtype=torch.float64, device=col.device), (n, n))


def _transposed(n, rp, col, wt):
    row = torch.repeat_interleave(torch.arange(n, device=col.device), (rp[1:] - rp[:-1]).to(torch.int64))
    order = torch.argsort(col.to(torch.int64) * n + row)
    irp = torch.zeros(n + 1, dtype=torch.int64, device=col.device)
    irp[1:] = torch.cumsum(torch.bincount(col.to(torch.int64), minlength=n), 0)
    return irp.to(torch.int32), row[order].to(torch.int32), None if wt is None else wt[order]


def _dependencies(n, A, At, src, lane, S):
    """Sum over the columns of delta (sources excluded): column lane[i] holds
    the traversal from src[i]; level by level with sparse products."""
    sig = torch.zeros(n, S, dtype=torch.float64, device=src.device)
    dist = torch.full((n, S), -1, dtype=torch.int32, device=src.device)
    sig[src, lane] = 1.0
    dist[src, lane] = 0
    level = 0
    while True:
        x = torch.sparse.mm(At, torch.where(dist == level, sig, 0.0))
        new = (x > 0) & (dist < 0)
        if not bool(new.any()):
            break
        level += 1
        dist[new] = level
        sig[new] = x[new]
    delta = torch.zeros_like(sig)
    for l in range(level, 0, -1):
        y = torch.sparse.mm(A, torch.where(dist == l, (1.0 + delta) / torch.where(dist == l, sig, 1.0), 0.0))
        delta = torch.where(dist == l - 1, sig * y, delta)
    delta[src, lane] = 0.0
    return delta.sum(1)


def _segment_sum(data, rp):
    return torch.segment_reduce(data, "sum", offsets=rp, axis=0, unsafe=True)


def _dependencies_weighted(n, out, inn, src, lane, S):
    """The same under arc weights: distances by relaxation to a fixed point,
    then path counts and dependencies by sweeps over the shortest-path arcs
    until they no longer change (the longest such path bounds the sweeps)."""
    (rp, col, wt), (irp, icol, iwt) = out, inn
    dist = torch.full((n, S), math.inf, dtype=torch.float64, device=src.device)
    dist[src, lane] = 0.0
    while True:
        best = torch.segment_reduce(dist[icol] + iwt[:, None], "min", offsets=irp, axis=0, unsafe=True, initial=math.inf)
        best = torch.minimum(best, dist)
        if torch.equal(best, dist):
            break
        dist = best
    rows = torch.repeat_interleave(torch.arange(n, device=src.device), rp[1:] - rp[:-1])
    irows = torch.repeat_interleave(torch.arange(n, device=src.device), irp[1:] - irp[:-1])
    on_in = (dist[icol] + iwt[:, None] == dist[irows]) & torch.isfinite(dist[irows])
    start = torch.zeros_like(dist)
    start[src, lane] = 1.0
    sig = start
    while True:
        nxt = start + _segment_sum(torch.where(on_in, sig[icol], 0.0), irp)
        if torch.equal(nxt, sig):
            break
        sig = nxt
    del on_in, irows
    on_out = (dist[rows] + wt[:, None] == dist[col]) & torch.isfinite(dist[rows])
    safe = torch.where(sig > 0, sig, 1.0)
    delta = torch.zeros_like(sig)
    while True:
        nxt = sig * _segment_sum(torch.where(on_out, ((1.0 + delta) / safe)[col], 0.0), rp)
        if torch.equal(nxt, delta):
            break
        delta = nxt
    delta[src, lane] = 0.0
    return delta.sum(1)


def exact(case, seed):
    if case["kind"] == "policy_grad":
        w, X, Y, mask = (t.double() for t in _grad_inputs(case, seed))
        h, i, o = 32, b.BC_MLP_IN, b.BC_MLP_OUT
        w.requires_grad_(True)
        W1, b1, W2, b2, W3, b3 = torch.split(w, [h * i, h, h * h, h, o * h, o])
        y = torch.relu(X @ W1.view(h, i).T + b1)
        y = torch.relu(y @ W2.view(h, h).T + b2)
        y = y @ W3.view(o, h).T + b3
        loss = (mask * (y - Y) ** 2).sum() / (2 * mask.sum())
        loss.backward()
        return {"loss": loss.detach().view(1), "grad": w.grad}
    rp, col, wt, off, srcs = _inputs(case, seed)
    n = rp.numel() - 1
    s = torch.from_numpy(srcs.astype(np.int64)).cuda()
    # the column of every source: one each, or one per position in its graph of a union
    lane = torch.arange(s.numel(), device="cuda")
    if off is not None:
        first = np.searchsorted(srcs, off[:-1])
        lane -= torch.from_numpy(first[np.searchsorted(off, srcs, side="right") - 1]).cuda()
    it = _transposed(n, rp, col, wt) if case.get("directed") else (rp, col, wt)
    S = 32 if wt is not None else 64
    if wt is None:
        A = _sparse(rp, col)
        At = _sparse(it[0], it[1]) if case.get("directed") else A
    else:
        out, inn = ([t.to(torch.int64) for t in x] for x in ((rp, col, wt), it))
    total = torch.zeros(n, dtype=torch.float64, device="cuda")
    for k in range(0, int(lane.max()) + 1, S):
        sel = (lane >= k) & (lane < k + S)
        if wt is None:
            total += _dependencies(n, A, At, s[sel], lane[sel] - k, S)
        else:
            total += _dependencies_weighted(n, out, inn, s[sel], lane[sel] - k, S)
    return total
