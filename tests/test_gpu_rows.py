"""The pull programs' row classes against the oracle: rows of exactly the
lengths at which a row goes to more lanes (8, 32, 256 and 2,048 arcs) and their
neighbours, vertex counts around a workgroup's stretch, grids of one workgroup
up, thresholds fixed by the caller, renumbered graphs.  PageRank within 1e-6
relative L1 (FP32 ranks, compensated sums), until stable within its tolerance
plus 3e-6, beliefs within 1e-5 (an iteration is a contraction)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from paper_1812_04070_amd import gen
from tests.gpu_util import announce, rel_l1, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


EDGES = [1, 7, 8, 9, 31, 32, 33, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049]


def _rows(lengths, n, seed, directed):
    """Vertex k has lengths[k] neighbours among the others (in-arcs)."""
    r = np.random.default_rng(seed)
    e = []
    for v, d in enumerate(lengths):
        src = r.choice(np.arange(len(lengths), n), d, replace=False)
        e.append(np.stack([src, np.full(d, v)], axis=1))
        if directed and v % 3:
            e.append(np.stack([np.full(1, v), src[:1]], axis=1))
    e = np.concatenate(e)
    w = r.integers(1, 65, len(e))
    return gen.from_edges(n, e, w, directed=directed)


GRAPHS = [
    ("edges-5000", lambda d: _rows(EDGES, 5000, 1, d)),
    ("all-short-1025", lambda d: _rows([j % 9 + 1 for j in range(900)], 1025, 2, d)),
    ("one-wave-64", lambda d: _rows([3, 8, 20], 64, 3, d)),
    ("lanes-40961", lambda d: _rows([j % 300 + 1 for j in range(400)], 40961, 4, d)),
]
POLICIES = [("auto", sx.Policy()), ("one-workgroup", sx.Policy(grid_wgs=1)), ("three", sx.Policy(grid_wgs=3)),
            ("fixed-bins", sx.Policy(bin_small=4, bin_large=8)), ("wide-bins", sx.Policy(bin_small=128, bin_large=4096))]


@pytest.mark.parametrize("directed", [False, True], ids=["undirected", "directed"])
@pytest.mark.parametrize("name,make", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_pagerank_rows(engine, name, make, directed):
    g = make(directed)
    ref, fix = oracle.pagerank_g(g), oracle.pagerank_fixpoint_g(g, tol=1e-13)[0]
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        for pname, pol in POLICIES:
            announce(f"rows pagerank {name} directed={directed} reorder={reorder} {pname}")
            x, st = run(engine, g, sx.SX_PAGERANK, -1, pol, dg=dg)
            assert rel_l1(x, ref) <= 1e-6
            assert st["edges_inspected"] == 20 * g.m
            x, _ = run(engine, g, sx.SX_PAGERANK, -1, pol, dg=dg, pr_iters=0, pr_tol=1e-5)
            assert np.abs(x.astype(np.float64) - fix).sum() <= 1e-5 + 3e-6
        dg.close()


@pytest.mark.parametrize("name,make", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_bp_rows(engine, name, make):
    g = make(False)
    prior = gen.bp_priors(g.n, seed=5)
    for iters in (1, 2, 5):
        ref = oracle.bp_g(g, prior.astype(np.float64), 0.5, iters)
        for reorder in (False, True):
            dg = engine.load(g, reorder=reorder)
            for pname, pol in POLICIES:
                announce(f"rows bp {name} iters={iters} reorder={reorder} {pname}")
                b, _ = run(engine, g, sx.SX_BP, -1, pol, dg=dg, prior=prior, bp_kappa=0.5, bp_iters=iters)
                assert rel_l1(b, ref) <= 1e-5
            dg.close()
