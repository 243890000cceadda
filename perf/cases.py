"""The workloads whose time on the GPU is tracked: one pass of each ACC program
through the public entry points, over the range of graphs the engine serves.

A case names an algorithm, a graph recipe and the options of the call.  The
recipes are those of the evaluation workloads (R-MAT with a, b, c = 0.57, 0.19,
0.19 and edge factor 16; four-neighbour grids with a tenth of the edges
deleted; the mixed batch), drawn here on the GPU with torch so that several
inputs of a case can be made quickly.  ``n`` below ``2 ** scale`` keeps the
first n vertices of the R-MAT graph, so that vertex counts are not all powers
of two.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1812_04070_amd as sx

_ENGINE = None


def _engine() -> sx.Engine:
    global _ENGINE
    if _ENGINE is None:
        _ENGINE = sx.Engine(0)
    return _ENGINE


# ------------------------------------------------------------------ cases ---

def _rmat(name, algo, scale, **more):
    case = {"algo": algo, "graph": "rmat", "scale": scale, "n": 1 << scale, "edge_factor": 16, "directed": False,
            "weights": 64 if algo in ("sssp", "bp") else 0, "reorder": False, "source": "hub"}
    case.update(more)
    if name:
        case["name"] = name
    return case


def _grid(name, algo, side, **more):
    case = {"algo": algo, "graph": "grid", "side": side, "weights": 1000 if algo == "sssp" else 0,
            "reorder": False, "source": "hub"}
    case.update(more)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # a single query on a graph of a thousand vertices: launches and
        # latency, no work to speak of
        _rmat("bfs_rmat10", "bfs", 10),
        # the headline step: BFS, SSSP and the k-core decomposition of an
        # undirected social-network-like graph, renumbered at load
        _rmat("bfs_rmat22", "bfs", 22, reorder=True),
        _rmat("sssp_rmat22", "sssp", 22, reorder=True, delta="none"),
        _rmat("kcore_rmat22", "kcore", 22, reorder=True),
        # road-network-like graphs: thousands of levels of small frontiers
        _grid("bfs_grid2048", "bfs", 2048),
        _grid("sssp_grid4096", "sssp", 4096, delta="auto"),
        # connected components: the social-network graph and a mesh
        _rmat("wcc_rmat22", "wcc", 22, reorder=True),
        _grid("wcc_grid1024", "wcc", 1024),
        # PageRank of a directed graph: the fixed number of iterations at the
        # largest size, and until stable at a middle one
        _rmat("pagerank_rmat24d", "pagerank", 24, directed=True, reorder=True, iters=20),
        _rmat("pagerank_tol_rmat20d", "pagerank_tol", 20, directed=True, reorder=True, tol=1e-6),
        # belief propagation on a Markov random field over the social graph
        _rmat("bp_rmat22", "bp", 22, reorder=True, iters=10),
        # many BFS / SSSP queries over graphs of mixed kind and size
        {"name": "batch_48q", "algo": "batch", "n_rmat": 8, "n_grid": 2, "scale_lo": 12, "scale_hi": 17,
         "side_lo": 128, "side_hi": 512, "queries": 48, "team": 32},
    ]


def draw(rng: random.Random):
    algo = rng.choice(["bfs", "bfs", "sssp", "sssp", "kcore", "wcc", "pagerank", "pagerank_tol", "bp", "batch"])
    if algo == "batch":
        lo, side = rng.randint(10, 13), int(2 ** rng.uniform(5, 8))
        return {"algo": "batch", "n_rmat": rng.randint(2, 8), "n_grid": rng.randint(1, 2), "scale_lo": lo,
                "scale_hi": lo + rng.randint(1, 4), "side_lo": side, "side_hi": 2 * side,
                "queries": rng.randint(5, 48), "team": rng.choice([4, 16, 32])}
    if algo in ("bfs", "sssp", "wcc", "kcore") and rng.random() < 0.4:
        most = {"bfs": 11.0, "sssp": 12.0, "wcc": 10.0, "kcore": 11.0}[algo]
        side = int(2 ** rng.uniform(4.0, most))
        case = _grid(None, algo, side, source=rng.choice(["hub", "random"]))
        if algo == "sssp":
            # without buckets a grid's distances are corrected many times over
            case["delta"] = "none" if side <= 1024 and rng.random() < 0.5 else "auto"
        return case
    scale = rng.randint(8, 22)
    n = rng.choice([1 << scale, rng.randint((1 << (scale - 1)) + 1, 1 << scale)])
    case = _rmat(None, algo, scale, n=n, edge_factor=rng.choice([6, 8, 12, 16]),
                 reorder=rng.random() < 0.5, source=rng.choice(["hub", "random"]))
    if algo in ("bfs", "sssp", "kcore"):
        case["directed"] = rng.random() < 0.3
    if algo == "sssp":
        case["delta"] = rng.choice(["none", "auto"])
    if algo == "kcore":
        case["k"] = rng.choice([0, 0, 16])
    if algo == "pagerank":
        case.update(directed=rng.random() < 0.7, iters=rng.choice([5, 10, 20]))
    if algo == "pagerank_tol":
        case.update(directed=rng.random() < 0.7, tol=rng.choice([1e-4, 1e-5, 1e-6]))
    if algo == "bp":
        case.update(iters=rng.choice([3, 5, 10]), weights=rng.choice([0, 64]))
    return case


# ----------------------------------------------------------------- graphs ---

def _rng(seed: int) -> torch.Generator:
    return torch.Generator(device="cuda").manual_seed(seed)


def _csr(src, dst, n, w=None):
    """(offsets, indices, weights) of the arcs, rows sorted ascending."""
    key = src * n + dst
    if w is None:
        key, at = torch.sort(key)[0], None
    else:
        key, at = torch.sort(key)
    src = torch.div(key, n, rounding_mode="floor")
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(src, minlength=n), 0, out=off[1:])
    return off.to(torch.int32), (key - src * n).to(torch.int32), None if w is None else w[at]


def _rmat_edges(scale, n, edge_factor, gen, directed):
    """Unique edges (src, dst) without self loops among the first n vertices;
    src < dst unless directed."""
    count = edge_factor << scale
    u = torch.zeros(count, dtype=torch.int64, device="cuda")
    v = torch.zeros(count, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        r = torch.rand(count, generator=gen, device="cuda")
        bu = r >= 0.76
        bv = ((r >= 0.57) & ~bu) | (r >= 0.95)
        u.mul_(2).add_(bu)
        v.mul_(2).add_(bv)
    del r, bu, bv
    if not directed:
        u, v = torch.minimum(u, v), torch.maximum(u, v)
    key = torch.sort((u * n + v)[(u != v) & (u < n) & (v < n)])[0]
    del u, v
    keep = torch.ones_like(key, dtype=torch.bool)
    torch.ne(key[1:], key[:-1], out=keep[1:])
    key = key[keep]
    u = torch.div(key, n, rounding_mode="floor")
    return u, key - u * n


def _grid_edges(side, gen):
    at = torch.arange(side * side, device="cuda").view(side, side)
    u = torch.cat([at[:, :-1].reshape(-1), at[:-1].reshape(-1)])
    v = torch.cat([at[:, 1:].reshape(-1), at[1:].reshape(-1)])
    keep = torch.rand(u.numel(), generator=gen, device="cuda") >= 0.1
    return u[keep], v[keep]


def _graph(case, seed):
    """CSR (and, directed, CSC) tensors of the case's graph."""
    gen = _rng(seed)
    directed = bool(case.get("directed", False))
    if case["graph"] == "grid":
        n = case["side"] ** 2
        u, v = _grid_edges(case["side"], gen)
    else:
        n = case["n"]
        u, v = _rmat_edges(case["scale"], n, case["edge_factor"], gen, directed)
    w = None
    if case["weights"]:
        w = torch.randint(1, case["weights"] + 1, (u.numel(),), generator=gen, device="cuda", dtype=torch.int32)
    g = {"n": n, "directed": directed}
    if directed:
        g["off"], g["idx"], g["w"] = _csr(u, v, n, w)
        g["in_off"], g["in_idx"], g["in_w"] = _csr(v, u, n, w)
    else:
        g["off"], g["idx"], g["w"] = _csr(torch.cat([u, v]), torch.cat([v, u]), n,
                                          None if w is None else torch.cat([w, w]))
    return g


class Resident:
    """A graph in device memory, borrowed by the library."""

    def __init__(self, g, reorder=False):
        self.tensors = g
        self.n, self.m = g["n"], g["idx"].numel()
        flags = sx.SX_DEVICE_PTRS | (0 if g["directed"] else sx.SX_UNDIRECTED) | (sx.SX_REORDER if reorder else 0)
        ptr = [g[k].data_ptr() if g.get(k) is not None else None
               for k in ("off", "idx", "w", "in_off", "in_idx", "in_w")]
        torch.cuda.synchronize()
        self.handle = sx.sx_graph_load(_engine().ctx, sx.sx_graph_desc(self.n, self.m, *ptr, flags),
                                       _engine().stream())

    def __del__(self):
        if getattr(self, "handle", None):
            sx.sx_graph_destroy(self.handle)
            self.handle = None


def _source(g, how, gen):
    deg = g["off"][1:] - g["off"][:-1]
    if how == "hub":
        return int(torch.nonzero(deg == deg.max())[0])
    cand = torch.nonzero(deg > 0).view(-1)
    return int(cand[int(torch.randint(cand.numel(), (1,), generator=gen, device="cuda"))]) if cand.numel() else 0


def _priors(n, seed):
    return torch.rand(n, generator=_rng(seed + 77), device="cuda") * 0.8 + 0.1


# ------------------------------------------------------- prepare and run ---

def _prepare_batch(case, seed):
    r = random.Random(seed)
    gen = _rng(seed + 13)
    graphs = []
    for i in range(case["n_rmat"]):
        # scales and sides spread evenly over their range, so that inputs of
        # another seed are as much work
        s = case["scale_lo"] + i * (case["scale_hi"] - case["scale_lo"]) // max(case["n_rmat"] - 1, 1)
        graphs.append(Resident(_graph(_rmat(None, "sssp", s), r.randrange(1 << 30))))
    for i in range(case["n_grid"]):
        side = case["side_lo"] + i * (case["side_hi"] - case["side_lo"]) // max(case["n_grid"] - 1, 1)
        graphs.append(Resident(_graph(_grid(None, "sssp", side, weights=64), r.randrange(1 << 30))))
    queries, outs = [], []
    for k in range(case["queries"]):
        g = graphs[k % len(graphs)]
        outs.append(torch.empty(g.n, dtype=torch.int32, device="cuda"))
        algo = sx.SX_SSSP if (k // len(graphs) + k) % 2 else sx.SX_BFS
        queries.append((g.handle, algo, _source(g.tensors, "random", gen), outs[-1].data_ptr()))
    return {"algo": "batch", "graphs": graphs, "queries": queries, "outs": outs,
            "cfg": sx.sx_batch_config(case["team"], 0, 0)}


def prepare(case, seed):
    if case["algo"] == "batch":
        return _prepare_batch(case, seed)
    g = _graph(case, seed)
    state = {"algo": case["algo"], "graph": Resident(g, case["reorder"]), "case": case}
    if case["algo"] in ("bfs", "sssp"):
        state["source"] = _source(g, case["source"], _rng(seed + 13))
    if case["algo"] == "bp":
        state["prior"] = _priors(g["n"], seed)
    return state


def run(state):
    eng, algo = _engine(), state["algo"]
    if algo == "batch":
        sx.sx_run_batch(eng.ctx, state["queries"], cfg=state["cfg"], stream=eng.stream())
        return state["outs"]
    g, case = state["graph"], state["case"]
    if algo == "bfs":
        return eng.run(g, sx.SX_BFS, state["source"])[0]
    if algo == "sssp":
        return eng.run(g, sx.SX_SSSP, state["source"],
                       sssp_delta=sx.SX_DELTA_AUTO if case["delta"] == "auto" else 0)[0]
    if algo == "kcore":
        return eng.run(g, sx.SX_KCORE, kcore_k=case.get("k", 0))[0]
    if algo == "wcc":
        return eng.run(g, sx.SX_WCC)[0]
    if algo == "pagerank":
        return eng.run(g, sx.SX_PAGERANK, pr_iters=case["iters"])[0]
    if algo == "pagerank_tol":
        return eng.run(g, sx.SX_PAGERANK, pr_iters=0, pr_tol=case["tol"])[0]
    return eng.run(g, sx.SX_BP, prior=state["prior"], bp_iters=case["iters"])[0]


# ------------------------------------------------------------------- work ---

def _size(case):
    """(vertices, arcs) of the case's graph; R-MAT arcs before duplicates go."""
    if case["graph"] == "grid":
        return case["side"] ** 2, int(3.6 * case["side"] * (case["side"] - 1))
    n = case["n"]
    share = (n / (1 << case["scale"])) ** 1.5
    return n, int(share * (case["edge_factor"] << case["scale"]) * (1 if case["directed"] else 2))


def work(case):
    """Graph arrays in and vertex arrays out once (the iterated programs: once
    per iteration, the graph being larger than any cache)."""
    algo = case["algo"]
    if algo == "batch":
        mid = (case["scale_lo"] + case["scale_hi"]) / 2
        arcs, side = 32 * 2 ** mid, (case["side_lo"] + case["side_hi"]) / 2
        per = (case["n_rmat"] * (6 * arcs + 8 * 2 ** mid) + case["n_grid"] * (6 * 3.6 + 8) * side ** 2)
        return {"bytes": per * case["queries"] / (case["n_rmat"] + case["n_grid"]), "flops": 0}
    n, m = _size(case)
    if algo == "sssp":
        return {"bytes": 8 * m + 8 * n, "flops": 0}
    if algo == "kcore":
        return {"bytes": 4 * m * (2 if case.get("directed") else 1) + 8 * n, "flops": 0}
    if algo in ("bfs", "wcc"):
        return {"bytes": 4 * m + 8 * n, "flops": 0}
    if algo == "bp":
        return {"bytes": case["iters"] * (8 * m + 12 * n), "flops": case["iters"] * 6 * m}
    # a step contracts the change by the damping factor 0.85
    iters = case["iters"] if algo == "pagerank" else math.ceil(math.log(case["tol"]) / math.log(0.85) / 4)
    return {"bytes": iters * (4 * m + 12 * n), "flops": iters * m}


# ------------------------------------------------------------------ exact ---

def _row_sums(off, terms):
    """Sums of each row's terms, in 64 bits: differences of one prefix sum."""
    total = torch.cat([terms.new_zeros(1), torch.cumsum(terms, 0)])
    off = off.long()
    return total[off[1:]] - total[off[:-1]]


def _exact_pagerank(g, iters, tol):
    n, d = g["n"], 0.85
    outdeg = (g["off"][1:] - g["off"][:-1]).double()
    in_off, in_idx = (g["in_off"], g["in_idx"]) if g["directed"] else (g["off"], g["idx"])
    x = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    for _ in range(iters):
        c = torch.where(outdeg > 0, x / outdeg.clamp(min=1), torch.zeros_like(x))
        y = (1 - d) / n + d * (_row_sums(in_off, c[in_idx]) + x[outdeg == 0].sum() / n)
        moved = float((y - x).abs().sum())
        x = y
        if tol and moved <= tol:
            break
    return x


def _exact_bp(g, prior, iters, kappa=0.5):
    off, cols = g["off"], g["idx"]
    deg = (off[1:] - off[:-1]).double()
    theta = 1.0 if g["w"] is None else (((g["w"] - 1) & 63).double() - 31.5) / 31.5
    c = kappa * theta / torch.maximum(torch.repeat_interleave(deg, deg.long()), deg[cols])
    h = torch.atanh(2 * prior.double() - 1)
    x = h
    for _ in range(iters):
        x = h + _row_sums(off, torch.atanh(c * torch.tanh(x)[cols]))
    return torch.sigmoid(2 * x)


def exact(case, seed):
    if case["algo"] not in ("pagerank", "pagerank_tol", "bp"):
        return None
    g = _graph(case, seed)
    if case["algo"] == "bp":
        return _exact_bp(g, _priors(g["n"], seed), case["iters"])
    if case["algo"] == "pagerank":
        return _exact_pagerank(g, case["iters"], 0.0)
    return _exact_pagerank(g, 400, 1e-13)
