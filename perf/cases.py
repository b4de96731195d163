"""The measured workloads: what a user of this library has it do, as plain cases.

A case names a graph family with its sizes and one public entry point.  The
families and sizes are the benchmark's and the tests' (R-MAT, directed R-MAT,
uniform random, road-like grids with and without shortcuts, weighted R-MAT),
drawn here with torch on the device so that making an input is quick:

  one_source_small    one query source on a 4K-vertex resident graph: latency
                      and launch count
  all_sources_small   exact BC (every vertex a source) of the 4K-vertex R-MAT
  graphs_mix          one call over 16 small graphs of uneven size
  requests_shared     the serving path: queued requests of 1, 8 and 64 sources
                      on one resident mid-size graph, sharing batches
  one_source_large    one query source on a 1M-vertex graph, the smallest
                      request of the serving mix on a large graph
  batch_rmat          the headline: scale-22 R-MAT, 256 sampled sources
  batch_directed      a directed graph, a ragged number of sources
  batch_uniform       uniform random graph, an odd vertex count
  road_shortcuts      road-like grid with shortcuts: ~100 levels
  road_deep           the same at full diameter: >1,500 levels and path counts
                      beyond double's range; ragged grid and source count
  sssp_rmat           weighted shortest paths on the scale-22 R-MAT
  pagerank_rmat       PageRank iterations on the scale-22 R-MAT

`draw` spreads the same families, entry points and options over their sizes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2401_02472_amd as bcm

DEV = "cuda"


def listed():
    return [
        {"name": "one_source_small", "call": "bc", "graph": "rmat", "scale": 12, "ef": 8, "k": 1},
        {"name": "all_sources_small", "call": "bc", "graph": "rmat", "scale": 12, "ef": 8,
         "k": 4096},
        {"name": "graphs_mix", "call": "graphs", "graph": "rmat", "scale": 10, "ef": 16,
         "graphs": 16, "k": 64},
        {"name": "requests_shared", "call": "multi", "graph": "rmat", "scale": 16, "ef": 16,
         "k": 154},
        {"name": "one_source_large", "call": "bc", "graph": "rmat", "scale": 20, "ef": 16, "k": 1},
        {"name": "batch_rmat", "call": "bc", "graph": "rmat", "scale": 22, "ef": 16, "k": 256},
        {"name": "batch_directed", "call": "bc", "graph": "rmat_dir", "scale": 20, "ef": 16,
         "k": 100},
        {"name": "batch_uniform", "call": "bc", "graph": "uniform", "n": 4000037, "deg": 16,
         "k": 128},
        {"name": "road_shortcuts", "call": "bc", "graph": "grid", "rows": 1024, "cols": 1024,
         "short": 0.001, "k": 64},
        {"name": "road_deep", "call": "bc", "graph": "grid", "rows": 1019, "cols": 997,
         "short": 0.0, "k": 50},
        {"name": "sssp_rmat", "call": "sssp", "graph": "rmat", "scale": 22, "ef": 16},
        {"name": "pagerank_rmat", "call": "pagerank", "graph": "rmat", "scale": 22, "ef": 16,
         "tol": 0.0, "iters": 20},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same families and entry points, sizes spread over
    their logarithms (k * arcs at most the headline's)."""
    call = rng.choice(["bc", "bc", "bc", "bc", "multi", "graphs", "sssp", "pagerank"])
    if call == "graphs":
        return {"call": "graphs", "graph": "rmat", "scale": rng.randint(8, 13),
                "ef": rng.randint(4, 16), "graphs": rng.randint(2, 24), "k": _log(rng, 4, 300)}
    if call == "multi":
        return {"call": "multi", "graph": "rmat", "scale": rng.randint(12, 20),
                "ef": rng.randint(8, 16), "k": _log(rng, 3, 300)}
    fam = rng.choice({"bc": ["rmat", "rmat", "rmat_dir", "uniform", "grid", "grid"],
                      "sssp": ["rmat", "rmat", "uniform", "grid"],
                      "pagerank": ["rmat", "rmat_dir", "uniform"]}[call])
    if fam == "uniform":
        case = {"call": call, "graph": fam, "n": _log(rng, 1000, 3000000), "deg": rng.randint(3, 20)}
    elif fam == "grid":
        case = {"call": call, "graph": fam, "rows": _log(rng, 24, 700), "cols": _log(rng, 24, 700),
                "short": rng.choice([0.001, 0.001, 0.0])}
    else:
        case = {"call": call, "graph": fam, "scale": rng.randint(9, 21), "ef": rng.randint(4, 16)}
    if call == "bc":
        case["k"] = _log(rng, 1, 400) if fam != "grid" else _log(rng, 16, 130)
    elif call == "pagerank":
        case["tol"] = rng.choice([0.0, 1e-10])
        case["iters"] = rng.randint(5, 60)
    return case


# ---- inputs -----------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _csr(n, u, v, directed):
    """Device CSR of the arcs (both directions unless directed), loops and
    duplicates removed."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = u * n + v
    if not directed:
        key = torch.cat([key, v * n + u])
    key = torch.unique(key)
    src = torch.div(key, n, rounding_mode="floor")
    col = (key - src * n).to(torch.int32)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    return rp.to(torch.int32).contiguous(), col.contiguous()


def _rmat(scale, ef, gen, directed):
    n = 1 << scale
    m = ef * n
    u = torch.zeros(m, dtype=torch.int64, device=DEV)
    v = torch.zeros(m, dtype=torch.int64, device=DEV)
    for _ in range(scale):  # quadrants 0.57, 0.19, 0.19, 0.05
        r = torch.rand(m, generator=gen, device=DEV)
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    perm = torch.randperm(n, generator=gen, device=DEV)
    return (n,) + _csr(n, perm[u], perm[v], directed)


def _uniform(n, deg, gen):
    m = n * deg // 2
    u = torch.randint(n, (m,), generator=gen, device=DEV)
    v = torch.randint(n, (m,), generator=gen, device=DEV)
    return (n,) + _csr(n, u, v, False)


def _grid(rows, cols, short, gen):
    n = rows * cols
    at = torch.arange(n, device=DEV).view(rows, cols)
    u = torch.cat([at[:, :-1].reshape(-1), at[:-1].reshape(-1)])
    v = torch.cat([at[:, 1:].reshape(-1), at[1:].reshape(-1)])
    keep = torch.rand(u.numel(), generator=gen, device=DEV) >= 0.05
    u, v = u[keep], v[keep]
    extra = int(round(short * u.numel()))
    if extra:
        u = torch.cat([u, torch.randint(n, (extra,), generator=gen, device=DEV)])
        v = torch.cat([v, torch.randint(n, (extra,), generator=gen, device=DEV)])
    return (n,) + _csr(n, u, v, False)


def _graph(case, gen, step=0):
    """(n, row_ptr, col_idx) on the device; graph `step` of a case of several."""
    fam = case["graph"]
    if fam == "uniform":
        return _uniform(case["n"], case["deg"], gen)
    if fam == "grid":
        return _grid(case["rows"], case["cols"], case["short"], gen)
    return _rmat(case["scale"] + step % 3, case["ef"], gen, fam == "rmat_dir")


def _sources(n, rp, k, gen):
    """k distinct sources of degree >= 1 (all vertices when k >= n: exact BC)."""
    if k >= n:
        return np.arange(n, dtype=np.int32)
    cand = torch.nonzero(rp[1:] > rp[:-1]).view(-1)
    pick = torch.randperm(cand.numel(), generator=gen, device=DEV)[:k]
    return cand[pick].to(torch.int32).cpu().numpy()


def _weights(n, rp, ci, gen):
    """One weight in [1, 100] per edge, the same on both of its arcs."""
    salt = int(torch.randint(1 << 30, (1,), generator=gen, device=DEV).item())
    src = torch.repeat_interleave(torch.arange(n, device=DEV), (rp[1:] - rp[:-1]).long())
    a, b = torch.minimum(src, ci.long()), torch.maximum(src, ci.long())
    h = (a * 2654435761 + b * 40503 + salt) & 0x7FFFFFFF
    h = ((h ^ (h >> 15)) * 73244475) & 0x7FFFFFFF
    h = ((h ^ (h >> 13)) * 73244475) & 0x7FFFFFFF
    return ((h ^ (h >> 16)) % 100 + 1).to(torch.int32).cpu().numpy()


def _requests(k, src):
    """Requests of 1, 8 and 64 sources in turn, the last one ragged."""
    out, at, i = [], 0, 0
    while at < k:
        m = min((1, 8, 64)[i % 3], k - at)
        out.append(src[at:at + m])
        at += m
        i += 1
    return out


def _inputs(case, seed):
    """The arrays of a case, the same for prepare and exact."""
    gen = _gen(seed)
    many = case["graphs"] if case["call"] == "graphs" else 1
    graphs = [_graph(case, gen, i) for i in range(many)]
    srcs = [_sources(n, rp, case.get("k", 1), gen) for n, rp, _ in graphs]
    return graphs, srcs, gen


def prepare(case, seed):
    graphs, srcs, gen = _inputs(case, seed)
    flags = bcm.BC_GRAPH_INPUT_ON_DEVICE
    flags |= bcm.BC_GRAPH_DIRECTED if case["graph"] == "rmat_dir" else bcm.BC_GRAPH_TRUST_SYMMETRIC
    handles = [bcm.Graph(n, rp, ci, flags) for n, rp, ci in graphs]
    state = {"call": case["call"], "graphs": handles, "sources": srcs}
    n = graphs[0][0]
    if case["call"] == "sssp":
        handles[0].set_weights(_weights(*graphs[0], gen))
        state["dist"] = torch.empty(n, dtype=torch.int32, device=DEV)
    elif case["call"] == "pagerank":
        state["pr"] = torch.empty(n, dtype=torch.float64, device=DEV)
        state["tol"], state["iters"] = case["tol"], case["iters"]
    elif case["call"] == "multi":
        state["requests"] = _requests(len(srcs[0]), srcs[0])
        state["outs"] = [torch.empty(n, dtype=torch.float64, device=DEV)
                         for _ in state["requests"]]
    else:
        state["outs"] = [torch.empty(g.n, dtype=torch.float64, device=DEV) for g in handles]
    return state


def run(state):
    call, graphs = state["call"], state["graphs"]
    if call == "bc":
        graphs[0].run_async(state["sources"][0], state["outs"][0])
        return state["outs"][0]
    if call == "multi":
        graphs[0].run_multi(state["requests"], state["outs"])
        return state["outs"]
    if call == "graphs":
        bcm.bc_run_graphs(graphs, state["sources"], state["outs"])
        return state["outs"]
    if call == "sssp":
        return graphs[0].sssp(int(state["sources"][0][0]), state["dist"])
    pr, it = graphs[0].pagerank(0.85, state["tol"], state["iters"], state["pr"])
    return {"pr": pr, "iterations": it}


# ---- work and exact values ----------------------------------------------------


def _size(case, step=0):
    """(vertices, arcs) of graph `step`, without the few duplicates' removal."""
    fam = case["graph"]
    if fam == "uniform":
        return case["n"], case["n"] * case["deg"]
    if fam == "grid":
        return case["rows"] * case["cols"], int(3.8 * case["rows"] * case["cols"])
    n = 1 << (case["scale"] + step % 3)
    return n, case["ef"] * n * (1 if fam == "rmat_dir" else 2)


def work(case):
    """The CSR read once and each output written once; BC: an addition per arc
    and source in each of the two passes; PageRank: one per arc and iteration."""
    call = case["call"]
    total, flops = 0, 0
    for i in range(case["graphs"] if call == "graphs" else 1):
        n, m = _size(case, i)
        k = min(case.get("k", 1), n)
        total += 4 * (n + 1) + 4 * m
        if call == "sssp":
            total += 4 * m + 4 * n
            flops += m
        elif call == "pagerank":
            # 0 tolerance runs them all; else at least a few tens are needed
            its = case["iters"] if case["tol"] == 0 else min(case["iters"], 20)
            total += 8 * n
            flops += 2 * m * its
        else:
            outs = len(_requests(k, np.zeros(k))) if call == "multi" else 1
            total += 8 * n * outs + 4 * k
            flops += 2 * m * k
    return {"bytes": total, "flops": flops}


def _brandes(n, rp, ci, sources):
    """Brandes' dependencies per source, [n, k] float64, in plain torch: level
    masks over all arcs, a group of sources at a time."""
    src = torch.repeat_interleave(torch.arange(n, device=DEV), (rp[1:] - rp[:-1]).long())
    dst = ci.long()
    m = max(int(dst.numel()), 1)
    out = []
    s_all = torch.as_tensor(sources, device=DEV).long()
    step = int(max(1, min(128, (1 << 27) // max(m, n))))
    for at in range(0, len(sources), step):
        s = s_all[at:at + step]
        lanes = torch.arange(len(s), device=DEV)
        dist = torch.full((n, len(s)), -1, dtype=torch.int32, device=DEV)
        sigma = torch.zeros(n, len(s), dtype=torch.float64, device=DEV)
        dist[s, lanes] = 0
        sigma[s, lanes] = 1.0
        level = 0
        while True:
            front = torch.where(dist == level, sigma, 0.0)
            new = torch.zeros_like(sigma).index_add_(0, dst, front[src])
            hit = (new > 0) & (dist < 0)
            if not bool(hit.any()):
                break
            level += 1
            dist[hit] = level
            sigma = torch.where(hit, new, sigma)
        delta = torch.zeros_like(sigma)
        for lv in range(level, 0, -1):
            c = torch.where(dist == lv, (1.0 + delta) / sigma, 0.0)
            up = torch.zeros_like(sigma).index_add_(0, src, c[dst])
            delta = torch.where(dist == lv - 1, sigma * up, delta)
        delta[s, lanes] = 0.0
        out.append(delta)
    return out


def exact(case, seed):
    """The same outputs in plain float64 torch; None where that takes too long
    (or, on the deepest grids, where counts pass float64's range)."""
    call = case["call"]
    if call == "sssp":
        return None  # whole numbers
    sizes = [_size(case, i) for i in range(case["graphs"] if call == "graphs" else 1)]
    if call == "pagerank":
        (n, rp, ci), = _inputs(case, seed)[0]
        deg = (rp[1:] - rp[:-1]).double()
        src = torch.repeat_interleave(torch.arange(n, device=DEV), (rp[1:] - rp[:-1]).long())
        dst = ci.long()
        pr = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
        its = 0
        for its in range(1, case["iters"] + 1):
            share = torch.where(deg > 0, pr / deg, 0.0)
            nxt = (1.0 - 0.85) / n + 0.85 * torch.zeros_like(pr).index_add_(0, dst, share[src])
            change = float((nxt - pr).abs().sum())
            pr = nxt
            if change <= case["tol"]:
                break
        return {"pr": pr, "iterations": its}
    deep = case["graph"] == "grid"
    cost = sum(m * min(case["k"], n) for n, m in sizes) * (12.0 if deep else 1.0)
    if cost > 4e9 or (deep and case["short"] == 0.0 and case["rows"] + case["cols"] > 700):
        return None
    graphs, srcs, _ = _inputs(case, seed)
    if call == "multi":
        parts = _brandes(*graphs[0], srcs[0])
        delta = torch.cat(parts, 1)
        outs, at = [], 0
        for r in _requests(len(srcs[0]), srcs[0]):
            outs.append(delta[:, at:at + len(r)].sum(1))
            at += len(r)
        return outs
    outs = [sum(d.sum(1) for d in _brandes(*g, s)) for g, s in zip(graphs, srcs)]
    return outs if call == "graphs" else outs[0]
