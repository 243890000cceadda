#!/usr/bin/env python3
"""Benchmark: BFS + SSSP + k-core decomposition on an undirected R-MAT scale-22
graph (edge factor 16, a=0.57 b=0.19 c=0.19 d=0.05, uint32 weights in [1,64]),
source = the vertex of highest degree.

One step = BFS and SSSP from the source and the full k-core decomposition,
each a separate run of the engine through the C ABI, with the graph already
resident in HBM (loaded with the library's degree-ordered renumbering,
SX_REORDER: sources and results stay in the generator's numbering, and the
per-run mapping of the result is inside the timed region).  Outputs are
checked bit for bit against the CPU oracle after the timed region; a
mismatch makes the run exit with status 1.

    python bench.py [--gpus 1] [--steps K] [--warmup W]

Prints one JSON line.  value = GTEPS of BFS and SSSP, the metric's own
figure: twice the source component's undirected edges (Graph500 count, once
per traversal) over the BFS plus SSSP device time of a step (HIP events
around each run on its stream; median over the timed steps).  The k-core
decomposition's time and the whole step's wall-clock time are separate
fields; `roofline` is for the step's dominant kernel (k-core's phase
kernel), with the algorithmic bytes counted the way the work statement
defines them (8 B per arc of a removed vertex + 4n B per level scan).
"""
from __future__ import annotations

import argparse
import json
import os
import platform
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=64)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--scale", type=int, default=22, help=argparse.SUPPRESS)
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle leg")
    ap.add_argument("--fused", type=int, default=0, help="0 auto, 1 fused, 2 unfused, 3 sequenced")
    ap.add_argument("--no-batch", action="store_true", help="skip the batched / learned-policy leg")
    ap.add_argument("--pagerank", action="store_true",
                    help="instead of the step: time PageRank (pull, FP32, 20 iterations) and the "
                         "k-core decomposition on the directed R-MAT scale 24 graph and print "
                         "their own JSON line")
    ap.add_argument("--grid", action="store_true",
                    help="instead of the step: time BFS + SSSP on the 4096 x 4096 grid with 10%% of "
                         "its edges deleted and print their own JSON line")
    ap.add_argument("--bp", action="store_true",
                    help="instead of the step: time belief propagation (10 iterations, kappa 0.5) on "
                         "the R-MAT scale 22 graph and print its own JSON line")
    ap.add_argument("--wcc", action="store_true",
                    help="instead of the step: time connected components (minimum-label propagation) on "
                         "the R-MAT scale 22 graph and print its own JSON line")
    ap.add_argument("--ablation", action="store_true",
                    help="instead of the step: time every kernel arrangement (no fusion, the sequenced "
                         "launches, selective fusion, all fusion) per algorithm on the R-MAT scale 22 "
                         "graph and the 4096^2 grid, with the register use of each kernel, and print "
                         "one JSON line")
    ap.add_argument("--delta", type=int, default=-1,
                    help="SSSP delta-stepping bucket width (0 = none; default: the workload's own)")
    ap.add_argument("--copy-calib", type=int, default=0, metavar="MIB",
                    help="only run a plain device copy of MIB MiB ten times (scales the HBM "
                         "byte counters of a profiler run) and exit")
    return ap.parse_args()


TRAFFIC_FILE = os.path.join(ROOT, "profiles", "kcore_seq_rmat22_hbm_traffic.json")
KERNEL_SOURCES = ["sx_kcore.hip", "sx_frontier.hpp", "sx_device.hpp", "sx_types.hpp"]


def kernel_source_hash() -> str:
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_1812_04070_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(kname: str):
    """HBM bytes per launch of `kname` from the committed profiler counters
    (FETCH_SIZE + WRITE_SIZE per dispatch, scaled by the same counters of a
    plain copy), or None when they were taken on other kernel sources or
    another kernel."""
    try:
        with open(TRAFFIC_FILE) as f:
            t = json.load(f)
    except OSError:
        return None
    if t.get("kernel") != kname or t.get("source_hash") != kernel_source_hash():
        return None
    return t.get("bytes_per_launch")


def copy_calib(mib: int):
    import torch
    n = mib << 20
    a = torch.empty(n, dtype=torch.uint8, device="cuda")
    b = torch.empty_like(a)
    a.fill_(1)
    torch.cuda.synchronize()
    for _ in range(10):
        b.copy_(a)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_read": n, "copy_bytes_written": n, "copies": 10}))


def algo_bytes(kind: str, st: dict, n: int, reached: int) -> float:
    """Algorithmic HBM bytes of the executed schedule (4-byte words, no
    cache-line rounding), from the engine's own counters:
      BFS   8 B per expanded worklist entry (row offsets) + 8 B per inspected
            arc (neighbour id + its state) + 12 B per reached vertex (state
            write, list write and read) + 4n B per metadata scan
      SSSP  8 B per expansion + 12 B per inspected arc (id, weight, distance)
            + 12 B per expansion (relaxation write, list write and read)
            + 4n B per metadata scan
      k-core 8 B per inspected arc (id + degree decrement, or id + stamp in a
            pull step) + 12 B per alive-list entry scanned (entry, core number,
            degree) + 16 B per vertex (core number and stamp writes, list
            write and read)
      WCC   8 B per expansion + 8 B per inspected arc (id, label) + 12 B per
            expansion (label and stamp write, list write and read) + 4n B
            per metadata scan."""
    e, x = st["edges_inspected"], st["vertex_expansions"]
    scans = st["ballot_iters"] + st["pull_iters"]
    if kind == "bfs":
        return 8.0 * x + 8.0 * e + 12.0 * reached + 4.0 * n * scans
    if kind == "sssp":
        return 8.0 * x + 12.0 * e + 12.0 * x + 4.0 * n * scans
    if kind == "kcore":
        return 8.0 * e + 12.0 * st["scan_entries"] + 16.0 * n
    if kind == "wcc":
        return 8.0 * x + 8.0 * e + 12.0 * x + 4.0 * n * scans
    raise KeyError(kind)


def kcore_bytes_by_definition(st: dict, arcs_removed: int, n: int) -> float:
    """k-core algorithmic bytes as the work statement defines them: 8 B per
    arc of a removed vertex (neighbour id + degree decrement) + 4n B per
    level scan (the degree test over every vertex).  In the full
    decomposition every vertex is removed once, so the arc term is 8 B per
    arc of the graph (in- plus out-arcs for a directed graph)."""
    return 8.0 * arcs_removed + 4.0 * n * st["ballot_iters"]


def trav_kernel_name(kind: str, fused: int, arcs: int, n: int) -> str:
    """Name of the phase kernel a run of `kind` launches (graphs of 2^25 arcs
    or more and at least 8 arcs per vertex take the traversal kernel built
    for six wavefronts per SIMD)."""
    if fused == 2:
        return "unfused per-phase kernels"
    seq = fused in (0, 3)
    if kind == "wcc" and fused == 0:
        return "k_wcc_* (hooking)"
    if kind == "kcore":
        return "k_kcore_seq" if seq else "k_kcore_fused"
    if kind in ("bfs", "sssp") and fused == 0 and arcs < 8 * n:
        return "k_cascade"   # takes the run over from the phases
    ops = {"bfs": "BfsOps", "wcc": "WccOps"}.get(kind, "SsspOps")
    if not seq:
        return f"k_fused<{ops}>"
    return f"k_seq<{ops}, 6>" if arcs >= (1 << 25) and arcs >= 8 * n else f"k_seq<{ops}>"


def cpu_leg(g, src, ref_step_edges):
    import oracle
    t0 = time.perf_counter()
    d = oracle.bfs_g(g, src)
    t1 = time.perf_counter()
    x = oracle.sssp_g(g, src)
    t2 = time.perf_counter()
    c = oracle.kcore_g(g)
    t3 = time.perf_counter()
    trav = t2 - t0
    return {
        "value": ref_step_edges / trav / 1e9,
        "unit": "GTEPS",
        "cores": 1,
        "kind": "oracle",
        "sample": ("BFS + SSSP from the same source on the same R-MAT scale-22 graph (the value's "
                   "edges over their time), then the k-core decomposition: FIFO-queue BFS, binary-heap "
                   "Dijkstra and Batagelj-Zaversnik k-core, serial C -O2 on one host core; "
                   f"bfs {1e3*(t1-t0):.0f} ms, sssp {1e3*(t2-t1):.0f} ms, kcore {1e3*(t3-t2):.0f} ms; "
                   f"host: {platform.processor() or platform.machine()}, {os.cpu_count()} cpus visible"),
        "ms_bfs_sssp": 1e3 * trav,
        "ms_kcore": 1e3 * (t3 - t2),
    }, (d, x, c)


def batched_leg(eng, sx, gen, log, check=True):
    """256 BFS/SSSP queries over 64 graphs: sequential single-query runs with
    the heuristic policy against one batched launch (autotuned teams), with
    the heuristic and with the learned policy.  Results must be identical."""
    import torch
    t0 = time.perf_counter()
    graphs, queries = gen.batch_workload()
    log(f"[bench] batch workload: {len(graphs)} graphs, {len(queries)} queries, gen {time.perf_counter()-t0:.1f}s")
    dgs = [eng.load(g) for g in graphs]
    algo = {"bfs": sx.SX_BFS, "sssp": sx.SX_SSSP}
    outs_single = [torch.empty(graphs[gi].n, dtype=torch.int32, device=eng.device) for gi, _, _ in queries]
    outs_batch = [torch.empty(graphs[gi].n, dtype=torch.int32, device=eng.device) for gi, _, _ in queries]
    heur = sx.Policy()
    # single-query form, heuristic policy: one sx_run per query, back to back
    def singles():
        for (gi, a, s), o in zip(queries, outs_single):
            eng.run(dgs[gi], algo[a], s, heur, out=o)
    singles()
    torch.cuda.synchronize()
    log("[bench] batch: single-query warm-up done")
    reps = 1
    t0 = time.perf_counter()
    for _ in range(reps):
        singles()
    torch.cuda.synchronize()
    single_ms = 1e3 * (time.perf_counter() - t0) / reps
    log(f"[bench] batch: single-query form {single_ms:.1f} ms")
    qs = [(dgs[gi].handle, algo[a], s, o.data_ptr()) for (gi, a, s), o in zip(queries, outs_batch)]
    cfg, tune_ms = sx.sx_batch_autotune(eng.ctx, qs, heur.c(), eng.stream())
    log(f"[bench] autotuned batch config {cfg} ({tune_ms:.2f} ms)")

    def batch(pol):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            ms, _ = sx.sx_run_batch(eng.ctx, qs, pol, None, eng.stream())
        torch.cuda.synchronize()
        return 1e3 * (time.perf_counter() - t) / reps, ms

    batch_ms, batch_dev_ms = batch(heur.c())
    log(f"[bench] batch: batched form {batch_ms:.1f} ms")
    same = all(torch.equal(a, b) for a, b in zip(outs_single, outs_batch))
    res = {"graphs": len(graphs), "queries": len(queries), "single_query_ms": round(single_ms, 3),
           "batch_ms": round(batch_ms, 3), "batch_device_ms": round(batch_dev_ms, 3),
           "speedup_batched_vs_single": round(single_ms / batch_ms, 3), "team_config": cfg,
           "identical_to_single": bool(same)}
    params = load_trained_policy()
    if params is not None:
        sx.sx_policy_load_mlp(eng.ctx, params)
        lp = sx.Policy(policy=sx.SX_POLICY_LEARNED)
        lbatch_ms, _ = batch(lp.c())
        same_l = all(torch.equal(a, b) for a, b in zip(outs_single, outs_batch))
        # learned policy in the single-query form as well
        def singles_l():
            for (gi, a, s), o in zip(queries, outs_batch):
                eng.run(dgs[gi], algo[a], s, lp, out=o)
        singles_l()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(reps):
            singles_l()
        torch.cuda.synchronize()
        lsingle_ms = 1e3 * (time.perf_counter() - t0) / reps
        same_l = same_l and all(torch.equal(a, b) for a, b in zip(outs_single, outs_batch))
        res.update({"learned_batch_ms": round(lbatch_ms, 3), "learned_single_query_ms": round(lsingle_ms, 3),
                    "speedup_learned_batched_vs_heuristic_single": round(single_ms / lbatch_ms, 3),
                    "speedup_learned_vs_heuristic_single": round(single_ms / lsingle_ms, 3),
                    "learned_identical": bool(same_l)})
    if check:
        # the oracle on a sample of the queries (two of every eight, so that
        # BFS and SSSP queries alternate as in the workload; the full workload
        # is compared query by query in the GPU tests)
        import oracle
        t0 = time.perf_counter()
        sample = [qi for qi in range(len(queries)) if qi % 8 < 2]
        same_o = True
        for qi in sample:
            gi, a, s = queries[qi]
            ref = oracle.bfs_g(graphs[gi], s) if a == "bfs" else oracle.sssp_g(graphs[gi], s)
            same_o = same_o and np.array_equal(eng.to_host(dgs[gi], algo[a], outs_single[qi]), ref)
        res["bit_exact_vs_oracle"] = bool(same_o and same and res.get("learned_identical", True))
        res["oracle_checked_queries"] = len(sample)
        log(f"[bench] batch: oracle check of {len(sample)} queries in {time.perf_counter()-t0:.1f}s")
    for d in dgs:
        d.close()
    return res


def load_trained_policy():
    path = os.path.join(ROOT, "paper_1812_04070_amd", "policy_mlp.json")
    if not os.path.exists(path):
        return None
    with open(path) as f:
        return np.asarray(json.load(f)["params"], dtype=np.float32)


def pagerank_main(args):
    """PageRank on the directed R-MAT scale-24 graph (edge factor 16, deduped,
    no self loops): one run = 20 pull iterations in one persistent launch.
    Algorithmic bytes per iteration: 8 per arc (CSC neighbour id +
    contribution) + 20 per vertex (row offsets, out-degree, rank read and
    write, contribution write)."""
    import torch
    import paper_1812_04070_amd as sx
    from paper_1812_04070_amd import gen
    log = lambda s: print(s, file=sys.stderr, flush=True)
    t0 = time.perf_counter()
    g = gen.workload_graph("rmat24d", scale_override=args.scale if args.scale != 22 else None)
    log(f"[bench] graph rmat{args.scale if args.scale != 22 else 24}d: n={g.n} arcs={g.m} gen "
        f"{time.perf_counter()-t0:.1f}s")
    eng = sx.Engine(0)
    t0 = time.perf_counter()
    dg = eng.load(g, reorder=True)
    torch.cuda.synchronize()
    log(f"[bench] resident with degree-ordered renumbering in {time.perf_counter()-t0:.2f}s")
    out = torch.empty(g.n, dtype=torch.float32, device=eng.device)
    pol = sx.Policy()
    for _ in range(args.warmup):
        eng.run(dg, sx.SX_PAGERANK, -1, pol, out=out)
    torch.cuda.synchronize()
    dev = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        _, st = eng.run(dg, sx.SX_PAGERANK, -1, pol, out=out)
        dev.append(st["device_ms"])
    torch.cuda.synchronize()
    ms = 1e3 * (time.perf_counter() - t0) / args.steps
    iters = int(st["iterations"])
    dev_ms = float(np.median(dev))
    nbytes = (8.0 * g.m + 20.0 * g.n) * iters
    achieved = nbytes / (dev_ms / 1e3) / 1e9
    r = eng.to_host(dg, sx.SX_PAGERANK, out)
    # the k-core decomposition of the same graph (degree = in + out), timed
    # on its own after PageRank
    kout = torch.empty(g.n, dtype=torch.int32, device=eng.device)
    for _ in range(args.warmup):
        eng.run(dg, sx.SX_KCORE, -1, pol, out=kout)
    torch.cuda.synchronize()
    kdev = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        _, kst = eng.run(dg, sx.SX_KCORE, -1, pol, out=kout)
        kdev.append(kst["device_ms"])
    torch.cuda.synchronize()
    kms = 1e3 * (time.perf_counter() - t0) / args.steps
    kdev_ms = float(np.median(kdev))
    klaunch = max(1, int(kst["launches"]) - 1)
    kbytes = algo_bytes("kcore", kst, g.n, g.n)
    kc = eng.to_host(dg, sx.SX_KCORE, kout)
    log(f"[bench] k-core {kms:.2f} ms/run ({klaunch} phase launches)")
    kcore = {"ms": round(kms, 3), "device_ms": round(kdev_ms, 3), "gteps": round(g.m / (kms / 1e3) / 1e9, 3),
             "kernel": trav_kernel_name("kcore", 0, g.m, g.n), "launches": klaunch,
             "levels_scanned": kst["ballot_iters"], "peel_steps": kst["iterations"],
             "avg_launch_us": round(1e3 * kdev_ms / klaunch, 3),
             "achieved_GBs": round(kcore_bytes_by_definition(kst, 2 * g.m, g.n) / (kdev_ms / 1e3) / 1e9, 2),
             "bytes_definition": "8 B per arc of a removed vertex (in + out) + 4n B per level scan",
             "achieved_GBs_executed_schedule": round(kbytes / (kdev_ms / 1e3) / 1e9, 2)}
    result = {
        "metric": "PageRank pull FP32, directed R-MAT s24, 20 iterations",
        "value": round(ms, 3), "unit": "ms", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms, 3), "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": "rmat24d-pagerank", "n": g.n, "arcs": g.m, "iterations": iters,
                   "damping": 0.85, "reorder": True},
        "roofline": {"bound": "hbm", "kernel": "k_pr_fused", "achieved": round(achieved, 2),
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
                     "traffic": None, "launches": 1, "avg_launch_us": round(1e3 * dev_ms, 1),
                     "algorithmic_bytes_per_launch": nbytes},
    }
    # run until stable (Section 6): pull while most vertices change, then the
    # delta-accumulative push tail chosen by the decision tree
    tail = {}
    for tol in (1e-4, 1e-6):
        for _ in range(max(1, args.warmup)):
            eng.run(dg, sx.SX_PAGERANK, -1, pol, out=out, pr_tol=tol, pr_iters=0)
        tdev = []
        for _ in range(max(3, args.steps // 4)):
            _, tst = eng.run(dg, sx.SX_PAGERANK, -1, pol, out=out, pr_tol=tol, pr_iters=0)
            tdev.append(tst["device_ms"])
        tail[f"tol_{tol:g}"] = {"device_ms": round(float(np.median(tdev)), 3), "pull_iterations": tst["pull_iters"],
                                "push_steps": tst["iterations"] - tst["pull_iters"],
                                "arcs_inspected": tst["edges_inspected"]}
    log(f"[bench] pagerank until stable: {tail}")
    if not args.no_cpu:
        import oracle
        t0 = time.perf_counter()
        ref = oracle.pagerank_g(g)
        cpu_s = time.perf_counter() - t0
        result["rel_l1_vs_oracle"] = float(np.abs(r.astype(np.float64) - ref).sum() / np.abs(ref).sum())
        result["cpu_baseline"] = {"value": round(1e3 * cpu_s, 1), "unit": "ms", "cores": 1, "kind": "oracle",
                                  "sample": "the full 20-iteration FP64 PageRank of the same graph, serial C"}
        t0 = time.perf_counter()
        kref = oracle.kcore_g(g)
        kcore["oracle_ms"] = round(1e3 * (time.perf_counter() - t0), 1)
        kcore["bit_exact"] = bool(np.array_equal(kc, kref))
    else:
        result["cpu_baseline"] = None
    result["kcore"] = kcore
    result["until_stable"] = tail
    dg.close()
    eng.close()
    print(json.dumps(result))


def bp_main(args):
    """Belief propagation on the undirected R-MAT scale-22 graph (weights in
    [1, 64] give the couplings, priors uniform in [0.1, 0.9] from seed 22):
    one run = 10 synchronous sum-product iterations in one persistent
    launch.  Algorithmic bytes per iteration: 16 per arc (neighbour id,
    weight, the neighbour's 8-byte (q, degree) gather) + 20 per vertex (row
    offsets, prior field, new (q, degree))."""
    import torch
    import paper_1812_04070_amd as sx
    from paper_1812_04070_amd import gen
    log = lambda s: print(s, file=sys.stderr, flush=True)
    t0 = time.perf_counter()
    g = gen.workload_graph("rmat22")
    prior = gen.bp_priors(g.n, seed=22)
    log(f"[bench] graph rmat22: n={g.n} arcs={g.m} gen {time.perf_counter()-t0:.1f}s")
    eng = sx.Engine(0)
    dg = eng.load(g, reorder=True)
    dprior = torch.from_numpy(prior).to(eng.device)
    out = torch.empty_like(dprior)
    kappa, iters = 0.5, 10
    pol = sx.Policy()

    def once(it):
        out.copy_(dprior)
        return eng.run(dg, sx.SX_BP, -1, pol, out=out, bp_kappa=kappa, bp_iters=it)[1]

    for _ in range(args.warmup):
        once(iters)
    torch.cuda.synchronize()
    dev = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        dev.append(once(iters)["device_ms"])
    torch.cuda.synchronize()
    ms = 1e3 * (time.perf_counter() - t0) / args.steps
    dev_ms = float(np.median(dev))
    nbytes = (16.0 * g.m + 20.0 * g.n) * iters
    achieved = nbytes / (dev_ms / 1e3) / 1e9
    result = {
        "metric": "belief propagation FP32, R-MAT s22, 10 iterations",
        "value": round(ms, 3), "unit": "ms", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms, 3), "higher_is_better": False, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": "rmat22-bp", "n": g.n, "arcs": g.m, "iterations": iters, "kappa": kappa,
                   "reorder": True},
        "device_ms": {"median": round(dev_ms, 3), "mean": round(float(np.mean(dev)), 3),
                      "min": round(float(np.min(dev)), 3)},
        "roofline": {"bound": "hbm", "kernel": "k_bp_fused", "achieved": round(achieved, 2),
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
                     "traffic": None, "launches": 1, "avg_launch_us": round(1e3 * dev_ms, 1),
                     "algorithmic_bytes_per_launch": nbytes},
    }
    if not args.no_cpu:
        import oracle
        # bounded sample: two iterations on the same graph, device and oracle
        once(2)
        h = eng.to_host(dg, sx.SX_BP, out).astype(np.float64)
        t0 = time.perf_counter()
        ref = oracle.bp_g(g, prior.astype(np.float64), kappa, 2)
        cpu_s = time.perf_counter() - t0
        result["rel_l1_vs_oracle_2_iterations"] = float(np.abs(h - ref).sum() / np.abs(ref).sum())
        result["cpu_baseline"] = {"value": round(1e3 * cpu_s / 2 * iters, 1), "unit": "ms", "cores": 1,
                                  "kind": "oracle",
                                  "sample": "2 of the 10 iterations on the same graph (fp64, serial C), "
                                            "scaled to 10"}
    else:
        result["cpu_baseline"] = None
    dg.close()
    eng.close()
    print(json.dumps(result))


def wcc_main(args):
    """Connected components (minimum-label propagation, every vertex active
    at the start) on the undirected R-MAT scale-22 graph, renumbered;
    value = GTEPS over all undirected edges.  Labels are checked against the
    oracle's union-find after the timed region."""
    import torch
    import paper_1812_04070_amd as sx
    from paper_1812_04070_amd import gen
    log = lambda s: print(s, file=sys.stderr, flush=True)
    g = gen.workload_graph("rmat22")
    eng = sx.Engine(0)
    dg = eng.load(g, reorder=True)
    out = torch.empty(g.n, dtype=torch.int32, device=eng.device)
    pol = sx.Policy(fused=args.fused)
    for _ in range(args.warmup):
        eng.run(dg, sx.SX_WCC, -1, pol, out=out)
    torch.cuda.synchronize()
    dev = []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        _, st = eng.run(dg, sx.SX_WCC, -1, pol, out=out)
        dev.append(st["device_ms"])
    torch.cuda.synchronize()
    ms = 1e3 * (time.perf_counter() - t0) / args.steps
    dev_ms = float(np.median(dev))
    launches = max(1, int(st["launches"]) - 1)
    nbytes = algo_bytes("wcc", st, g.n, g.n)
    avg_us = 1e3 * dev_ms / launches
    achieved = nbytes / launches / (avg_us / 1e6) / 1e9
    lab = eng.to_host(dg, sx.SX_WCC, out)
    result = {
        "metric": "connected components (minimum labels), R-MAT s22", "value": round((g.m // 2) / (dev_ms / 1e3) / 1e9, 3),
        "unit": "GTEPS", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "int32", "data": "synthetic",
        "config": {"workload": "rmat22-wcc", "n": g.n, "arcs": g.m, "reorder": True},
        "device_ms": {"median": round(dev_ms, 4), "mean": round(float(np.mean(dev)), 4),
                      "min": round(float(np.min(dev)), 4)},
        "iterations": st["iterations"], "pull_iters": st["pull_iters"], "edges_inspected": st["edges_inspected"],
        "roofline": {"bound": "hbm", "kernel": trav_kernel_name("wcc", args.fused, g.m, g.n),
                     "achieved": round(achieved, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": None, "launches": launches,
                     "avg_launch_us": round(avg_us, 3), "algorithmic_bytes_per_launch": round(nbytes / launches, 1)},
    }
    if not args.no_cpu:
        import oracle
        t0 = time.perf_counter()
        ref = oracle.wcc_g(g)
        cpu_s = time.perf_counter() - t0
        result["bit_exact"] = bool(np.array_equal(lab, ref))
        result["cpu_baseline"] = {"value": round((g.m // 2) / cpu_s / 1e9, 4), "unit": "GTEPS", "cores": 1,
                                  "kind": "oracle", "sample": "union-find over the same graph, serial C"}
    else:
        result["cpu_baseline"] = None
    dg.close()
    eng.close()
    print(json.dumps(result))
    if result.get("bit_exact") is False:
        sys.exit(1)


def ablation_main(args):
    """Fusion ablation (Section 5, Table table-compile; Section 7,
    Fig. exp-selective-fusion): device time of each algorithm under each
    arrangement of the same phases -- none (one launch per phase, the host
    deciding in between), sequenced (one launch per phase, decisions on the
    device, launches queued ahead), selective fusion (one persistent kernel
    per direction, a direction change relaunches) and all fusion (one
    persistent kernel for both directions) -- where the engine has it, plus
    the kernels' registers and persistent grids.  Outputs of every arm are
    compared with the first arm's (bit for bit; PageRank and BP have one
    arrangement)."""
    import torch
    import paper_1812_04070_amd as sx
    from paper_1812_04070_amd import gen
    log = lambda s: print(s, file=sys.stderr, flush=True)
    eng = sx.Engine(0)
    arms = [("none", sx.SX_UNFUSED), ("sequenced", sx.SX_SEQUENCED), ("selective", sx.SX_FUSED),
            ("all", sx.SX_FUSED_ALL)]
    reps = max(3, min(args.steps, 7))
    table = {}
    for wname, reorder in (("rmat22", True), ("grid4096", False)):
        g = gen.workload_graph(wname)
        src = gen.max_degree_vertex(g)
        dg = eng.load(g, reorder=reorder)
        algos = [("bfs", sx.SX_BFS, src), ("sssp", sx.SX_SSSP, src), ("wcc", sx.SX_WCC, -1)]
        if wname == "rmat22":
            algos.append(("kcore", sx.SX_KCORE, -1))
        for aname, algo, s0 in algos:
            ref = None
            for arm, fused in arms:
                if aname == "kcore" and fused in (sx.SX_UNFUSED, sx.SX_FUSED_ALL):
                    continue       # k-core: sequenced launches or one persistent kernel
                pol = sx.Policy(fused=fused)
                kw = {"sssp_delta": sx.SX_DELTA_AUTO} if algo == sx.SX_SSSP else {}
                if wname == "grid4096" and fused == sx.SX_UNFUSED:
                    reps_here = 1  # thousands of host round trips
                else:
                    reps_here = reps
                ts = []
                for _ in range(reps_here + 1):
                    out, st = eng.run(dg, algo, s0, pol, **kw)
                    ts.append(st["device_ms"])
                h = eng.to_host(dg, algo, out)
                same = True if ref is None else bool(np.array_equal(h, ref))
                ref = h if ref is None else ref
                table[f"{wname}/{aname}/{arm}"] = {"ms": round(float(np.median(ts[1:])), 3),
                                                   "launches": st["launches"], "iterations": st["iterations"],
                                                   "barrier_wait_ms": round(st["barrier_wait_ms"], 3),
                                                   "same_as_first_arm": same}
                log(f"[ablation] {wname} {aname} {arm}: {table[f'{wname}/{aname}/{arm}']}")
        if wname == "rmat22":
            prior = gen.bp_priors(g.n, seed=22)
            for aname, algo, kw in (("bp", sx.SX_BP, {"prior": prior}),):
                ts = []
                for _ in range(reps + 1):
                    _, st = eng.run(dg, algo, -1, None, **kw)
                    ts.append(st["device_ms"])
                table[f"{wname}/{aname}/all"] = {"ms": round(float(np.median(ts[1:])), 3),
                                                 "launches": st["launches"], "iterations": st["iterations"]}
        dg.close()
    gd = gen.workload_graph("rmat24d")
    dgd = eng.load(gd, reorder=True)
    ts = []
    for _ in range(reps + 1):
        _, st = eng.run(dgd, sx.SX_PAGERANK, -1, None)
        ts.append(st["device_ms"])
    table["rmat24d/pagerank/all"] = {"ms": round(float(np.median(ts[1:])), 3), "launches": st["launches"],
                                     "iterations": st["iterations"]}
    dgd.close()
    regs = {}
    for k in ("bfs_fused", "bfs_fused_pull", "bfs_fused_all", "bfs_seq", "bfs_push_step", "bfs_pull_step",
              "sssp_fused", "sssp_fused_pull", "sssp_fused_all", "sssp_seq", "sssp_push_step",
              "sssp_pull_step", "wcc_fused", "wcc_fused_all", "wcc_seq", "kcore_fused", "kcore_seq",
              "pagerank_fused", "pagerank_until_stable", "pagerank_push_tail", "bp_fused", "batch"):
        regs[k] = eng.kernel_info(k)
    result = {"metric": "fusion ablation: device ms per algorithm and kernel arrangement", "value": None,
              "unit": "ms", "n_gpus": 1, "steps": reps, "warmup": 1, "higher_is_better": False,
              "data": "synthetic", "config": {"workload": "rmat22 (renumbered), grid4096, rmat24d"},
              "times": table, "kernels": regs}
    eng.close()
    print(json.dumps(result))


def grid_main(args):
    """BFS + SSSP on the 4096 x 4096 four-neighbour grid with 10 % of its
    edges deleted (weights in [1, 1000]) from the highest-degree vertex
    (ties to the lowest id): the high-diameter workload, thousands of small
    iterations.  Loaded without renumbering (grid ids already keep neighbours
    close).  value = GTEPS of the step (twice the source component's
    undirected edges over the step time)."""
    import torch
    import paper_1812_04070_amd as sx
    from paper_1812_04070_amd import gen
    log = lambda s: print(s, file=sys.stderr, flush=True)
    t0 = time.perf_counter()
    g = gen.workload_graph("grid4096")
    src = gen.max_degree_vertex(g)
    log(f"[bench] graph grid4096: n={g.n} arcs={g.m} src={src} gen {time.perf_counter()-t0:.1f}s")
    eng = sx.Engine(0)
    dg = eng.load(g)
    out_bfs = torch.empty(g.n, dtype=torch.int32, device=eng.device)
    out_sssp = torch.empty(g.n, dtype=torch.int32, device=eng.device)
    pol = sx.Policy(fused=args.fused)
    # the engine's own bucket width: 40 mean arc weights on a graph this
    # sparse, about 20,000 here (a sweep from 100 to 300,000 on this grid put
    # the best widths at 20,000-50,000: 215 ms against 619 without buckets)
    delta = args.delta if args.delta >= 0 else sx.SX_DELTA_AUTO

    def step():
        _, sb = eng.run(dg, sx.SX_BFS, src, pol, out=out_bfs)
        _, ss = eng.run(dg, sx.SX_SSSP, src, pol, out=out_sssp, sssp_delta=delta)
        return sb, ss

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    per = {"bfs": [], "sssp": []}
    t0 = time.perf_counter()
    for _ in range(args.steps):
        sb, ss = step()
        per["bfs"].append(sb)
        per["sssp"].append(ss)
        log(f"[bench] grid step done: bfs {sb['device_ms']:.2f} ms, sssp {ss['device_ms']:.2f} ms")
    torch.cuda.synchronize()
    ms_step = 1e3 * (time.perf_counter() - t0) / args.steps
    d = eng.to_host(dg, sx.SX_BFS, out_bfs)
    x = eng.to_host(dg, sx.SX_SSSP, out_sssp)
    deg = g.out_degree().astype(np.int64)
    m_cc = int(deg[d >= 0].sum() // 2)
    reached = int((d >= 0).sum())
    value = 2 * m_cc / (ms_step / 1e3) / 1e9
    algo_ms = {k: float(np.median([s["device_ms"] for s in v])) for k, v in per.items()}
    last = {k: v[-1] for k, v in per.items()}
    dom = max(algo_ms, key=algo_ms.get)
    nbytes = algo_bytes(dom, last[dom], g.n, reached)
    phase_launches = max(1, int(last[dom]["launches"]) - 1)
    avg_launch_us = 1e3 * algo_ms[dom] / phase_launches
    achieved = nbytes / phase_launches / (avg_launch_us / 1e6) / 1e9
    result = {
        "metric": "GTEPS BFS/SSSP on a 4096^2 grid (10% edges deleted), bit-exact",
        "value": round(value, 4), "unit": "GTEPS", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_step, 3), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "int32", "data": "synthetic",
        "config": {"workload": "grid4096-bfs-sssp", "side": 4096, "deleted": 0.1, "n": g.n, "arcs": g.m,
                   "source": src, "weights": [1, 1000], "m_cc": m_cc, "reached": reached, "reorder": False,
                   "sssp_delta": "auto" if delta == sx.SX_DELTA_AUTO else delta},
        "per_algo": {k: {"device_ms": round(algo_ms[k], 3), "iterations": last[k]["iterations"],
                         "launches": last[k]["launches"], "pull_iters": last[k]["pull_iters"],
                         "ballot_iters": last[k]["ballot_iters"], "edges_inspected": last[k]["edges_inspected"],
                         "vertex_expansions": last[k]["vertex_expansions"]} for k in per},
        "roofline": {"bound": "hbm", "kernel": trav_kernel_name(dom, args.fused, g.m, g.n),
                     "achieved": round(achieved, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 5), "traffic": None, "launches": phase_launches,
                     "avg_launch_us": round(avg_launch_us, 3),
                     "algorithmic_bytes_per_launch": round(nbytes / phase_launches, 1)},
    }
    if not args.no_cpu:
        import oracle
        log("[bench] cpu oracle leg")
        t0 = time.perf_counter()
        rd = oracle.bfs_g(g, src)
        t1 = time.perf_counter()
        rx = oracle.sssp_g(g, src)
        t2 = time.perf_counter()
        result["cpu_baseline"] = {
            "value": round(2 * m_cc / (t2 - t0) / 1e9, 5), "unit": "GTEPS", "cores": 1, "kind": "oracle",
            "sample": (f"one full step on the same grid: FIFO-queue BFS {1e3*(t1-t0):.0f} ms and binary-heap "
                       f"Dijkstra {1e3*(t2-t1):.0f} ms, serial C -O2 on one host core"),
            "ms_per_step": round(1e3 * (t2 - t0), 1)}
        result["bit_exact"] = bool(np.array_equal(d, rd) and np.array_equal(x, rx))
    else:
        result["cpu_baseline"] = None
    dg.close()
    eng.close()
    print(json.dumps(result))


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (asked for {args.gpus}): the engine has no multi-GPU "
              "path; the sharding design is described but not built.", file=sys.stderr)
        sys.exit(2)
    if args.copy_calib:
        copy_calib(args.copy_calib)
        return
    if args.pagerank:
        pagerank_main(args)
        return
    if args.grid:
        grid_main(args)
        return
    if args.bp:
        bp_main(args)
        return
    if args.ablation:
        ablation_main(args)
        return
    if args.wcc:
        wcc_main(args)
        return
    import torch
    import paper_1812_04070_amd as sx
    from paper_1812_04070_amd import gen
    log = lambda s: print(s, file=sys.stderr, flush=True)

    t_gen = time.perf_counter()
    g = gen.rmat(args.scale, 16, 0.57, 0.19, 0.19, seed=2, weights=(1, 64), weight_seed=102)
    src = gen.max_degree_vertex(g)
    t_gen = time.perf_counter() - t_gen
    log(f"[bench] graph rmat{args.scale}: n={g.n} arcs={g.m} src={src} gen {t_gen:.1f}s")

    eng = sx.Engine(0)
    dev = eng.device
    out_bfs = torch.empty(g.n, dtype=torch.int32, device=dev)
    out_sssp = torch.empty(g.n, dtype=torch.int32, device=dev)
    out_kc = torch.empty(g.n, dtype=torch.int32, device=dev)
    pol = sx.Policy(fused=args.fused)

    def step(dg):
        _, sb = eng.run(dg, sx.SX_BFS, src, pol, out=out_bfs)
        _, ss = eng.run(dg, sx.SX_SSSP, src, pol, out=out_sssp)
        _, sk = eng.run(dg, sx.SX_KCORE, -1, pol, out=out_kc)
        return sb, ss, sk

    def timed(dg, steps, warmup):
        for _ in range(warmup):
            step(dg)
        torch.cuda.synchronize()
        per = {"bfs": [], "sssp": [], "kcore": []}
        t0 = time.perf_counter()
        for _ in range(steps):
            sb, ss, sk = step(dg)
            per["bfs"].append(sb)
            per["sssp"].append(ss)
            per["kcore"].append(sk)
        torch.cuda.synchronize()
        return 1e3 * (time.perf_counter() - t0) / steps, per

    # the same step on the graph in the generator's numbering, for reference
    dg0 = eng.load(g)
    torch.cuda.synchronize()
    ms_plain, _ = timed(dg0, max(4, args.steps // 4), 1)
    dg0.close()
    log(f"[bench] step without renumbering: {ms_plain:.3f} ms")

    t_load = time.perf_counter()
    dg = eng.load(g, reorder=True)
    torch.cuda.synchronize()
    log(f"[bench] resident with degree-ordered renumbering in {time.perf_counter()-t_load:.2f}s")
    ms_step, per = timed(dg, args.steps, args.warmup)
    log(f"[bench] timed {args.steps} steps: {ms_step:.3f} ms/step")

    d = eng.to_host(dg, sx.SX_BFS, out_bfs)
    x = eng.to_host(dg, sx.SX_SSSP, out_sssp)
    c = eng.to_host(dg, sx.SX_KCORE, out_kc)
    deg = g.out_degree().astype(np.int64)
    m_cc = int(deg[d >= 0].sum() // 2)
    m_und = g.m // 2
    reached = int((d >= 0).sum())

    dev_ms = {k: np.array([s["device_ms"] for s in v]) for k, v in per.items()}
    algo_ms = {k: float(np.median(v)) for k, v in dev_ms.items()}
    trav = dev_ms["bfs"] + dev_ms["sssp"]
    trav_ms = float(np.median(trav))
    value = 2 * m_cc / (trav_ms / 1e3) / 1e9
    steps_dev = trav + dev_ms["kcore"]
    last = {k: v[-1] for k, v in per.items()}
    # dominant kernel: the kernel of the algorithm with the largest device
    # time.  Each run is one init launch followed by its phase launches, all
    # queued back to back on one stream, so the phase kernel's average launch
    # duration is the run's event-timed device time over its launch count
    # (rocprofv3 --kernel-trace --stats on the same command agrees: the
    # summaries under profiles/).
    dom = max(algo_ms, key=algo_ms.get)
    phase_launches = max(1, int(last[dom]["launches"]) - 1)
    avg_launch_us = 1e3 * algo_ms[dom] / phase_launches
    if dom == "kcore":
        nbytes = kcore_bytes_by_definition(last[dom], g.m, g.n)
        nbytes_exec = algo_bytes("kcore", last[dom], g.n, reached)
    else:
        nbytes = nbytes_exec = algo_bytes(dom, last[dom], g.n, reached)
    achieved = nbytes / phase_launches / (avg_launch_us / 1e6) / 1e9
    achieved_exec = nbytes_exec / phase_launches / (avg_launch_us / 1e6) / 1e9
    kname = trav_kernel_name(dom, args.fused, g.m, g.n)
    traffic = measured_traffic(kname)

    result = {
        "metric": "GTEPS BFS/SSSP R-MAT s22, bit-exact; learned-policy+batched vs heuristic speedup",
        "value": round(value, 3),
        "unit": "GTEPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "int32",
        "data": "synthetic",
        "config": {"workload": f"rmat{args.scale}-bfs-sssp-kcore", "scale": args.scale, "edge_factor": 16,
                   "n": g.n, "arcs": g.m, "source": src, "weights": [1, 64],
                   "m_cc": m_cc, "reached": reached, "reorder": True},
        "gteps_bfs": round(m_cc / (algo_ms["bfs"] / 1e3) / 1e9, 3),
        "gteps_sssp": round(m_cc / (algo_ms["sssp"] / 1e3) / 1e9, 3),
        "bfs_sssp_ms": {"median": round(trav_ms, 4), "mean": round(float(trav.mean()), 4),
                        "min": round(float(trav.min()), 4)},
        "kcore_ms": {"median": round(algo_ms["kcore"], 4), "mean": round(float(dev_ms["kcore"].mean()), 4),
                     "min": round(float(dev_ms["kcore"].min()), 4)},
        "step_device_ms": {"median": round(float(np.median(steps_dev)), 4),
                           "mean": round(float(steps_dev.mean()), 4), "min": round(float(steps_dev.min()), 4)},
        "step_gteps_incl_kcore": round((2 * m_cc + m_und) / (ms_step / 1e3) / 1e9, 3),
        "ms_per_step_without_renumbering": round(ms_plain, 4),
        "per_algo": {k: {"device_ms": round(algo_ms[k], 4),
                         "iterations": last[k]["iterations"], "launches": last[k]["launches"],
                         "pull_iters": last[k]["pull_iters"], "ballot_iters": last[k]["ballot_iters"],
                         "edges_inspected": last[k]["edges_inspected"],
                         "vertex_expansions": last[k]["vertex_expansions"],
                         "barrier_wait_ms": round(last[k]["barrier_wait_ms"], 4)} for k in per},
        "roofline": {"bound": "hbm", "kernel": kname, "achieved": round(achieved, 2),
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
                     "traffic": traffic,
                     "traffic_source": ("replayed: profiler counters (FETCH_SIZE, WRITE_SIZE, copy-calibrated) "
                                        "taken on the same kernel sources, not in this run"
                                        if traffic is not None else None),
                     "launches": phase_launches, "avg_launch_us": round(avg_launch_us, 3),
                     "algorithmic_bytes_per_launch": round(nbytes / phase_launches, 1),
                     "bytes_definition": ("8 B per arc of a removed vertex + 4n B per level scan"
                                          if dom == "kcore" else "executed schedule"),
                     "achieved_executed_schedule": round(achieved_exec, 2)},
    }
    if not args.no_batch:
        result["batched"] = batched_leg(eng, sx, gen, log, check=not args.no_cpu)
    ok = True
    if not args.no_cpu:
        log("[bench] cpu oracle leg")
        cpu, (rd, rx, rc) = cpu_leg(g, src, 2 * m_cc)
        result["cpu_baseline"] = cpu
        result["bit_exact"] = bool(np.array_equal(d, rd) and np.array_equal(x, rx) and np.array_equal(c, rc))
        ok = result["bit_exact"] and result.get("batched", {}).get("bit_exact_vs_oracle", True)
    else:
        result["cpu_baseline"] = None
    dg.close()
    eng.close()
    print(json.dumps(result))
    if not ok:
        log("[bench] outputs differ from the oracle")
        sys.exit(1)


if __name__ == "__main__":
    main()
