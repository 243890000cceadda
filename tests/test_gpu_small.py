"""BFS and SSSP runs that one workgroup takes as a whole (small graphs, default
policy) against the oracle: vertex counts around the bitmap word, the
workgroup and the limit, rows around the lengths a wavefront and the workgroup
take, more long rows in a frontier than their list holds, directed, renumbered
and no-allocation runs, unreachable vertices, distance overflow."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from paper_1812_04070_amd import gen
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


def _weighted(n, edges, seed, directed=False):
    w = np.random.default_rng(seed).integers(1, 65, len(edges))
    return gen.from_edges(n, edges, w, directed=directed)


def _random(n, m, seed, directed=False):
    return _weighted(n, np.random.default_rng(seed).integers(0, n, (m, 2)), seed, directed)


def _stars(lengths, n, seed):
    """Vertex 0 leads to vertices with rows of the given lengths."""
    r = np.random.default_rng(seed)
    e = [(0, k + 1) for k in range(len(lengths))]
    for k, d in enumerate(lengths):
        e += [(k + 1, int(u)) for u in r.choice(np.arange(len(lengths) + 1, n), d, replace=False)]
    return _weighted(n, e, seed, directed=True)


GRAPHS = [
    *[(f"random-{n}", lambda n=n: _random(n, 3 * n, n)) for n in (1, 2, 31, 32, 33, 1023, 1024, 1025)],
    ("directed-900", lambda: _random(900, 5000, 4, directed=True)),
    ("path-3000", lambda: _weighted(3000, [(i, i + 1) for i in range(2999)], 5)),
    ("rows", lambda: _stars([62, 63, 64, 65, 2046, 2047, 2048, 2049, 1], 9000, 6)),
    ("rows-1100-long", lambda: _stars([64 + k % 3 for k in range(1100)], 12000, 7)),
    ("grid-156", lambda: gen.grid(156, 0.1, seed=8, weights=(1, 64))),
    ("limit-24576", lambda: _random(24576, 45000, 9)),
    ("beyond-24577", lambda: _random(24577, 45000, 10)),
]


@pytest.mark.parametrize("name,make", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_small_exact(engine, name, make):
    g = make()
    one = g.n <= 24576
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        for s in sorted({0, g.n // 2, g.n - 1}):
            ref = oracle.bfs_g(g, s)
            announce(f"small bfs {name} reorder={reorder} src={s}")
            out, st = engine.run(dg, sx.SX_BFS, s)
            np.testing.assert_array_equal(engine.to_host(dg, sx.SX_BFS, out), ref)
            assert st["iterations"] == ref.max() + 1
            if one and g.m <= 1 << 17:
                assert st["launches"] == 1
            ref = oracle.sssp_g(g, s)
            announce(f"small sssp {name} reorder={reorder} src={s}")
            out, st = engine.run(dg, sx.SX_SSSP, s)
            np.testing.assert_array_equal(engine.to_host(dg, sx.SX_SSSP, out), ref)
            if one and g.m <= max(1 << 16, 4 * g.n):
                assert st["launches"] == 1
                again, st2 = engine.run(dg, sx.SX_SSSP, s)
                assert st2["iterations"] == st["iterations"]
            if not reorder:
                announce(f"small static {name} src={s}")
                out, _ = engine.run_static(dg, sx.SX_SSSP, s)
                np.testing.assert_array_equal(engine.to_host(dg, sx.SX_SSSP, out), ref)
        dg.close()


def test_small_overflow(engine):
    p = gen.from_edges(40, [(i, i + 1) for i in range(39)], [1 << 28] * 39)
    dg = engine.load(p)
    announce("small overflow")
    with pytest.raises(sx.SxError) as ei:
        engine.run(dg, sx.SX_SSSP, 0)
    assert ei.value.status == sx.SX_EOVERFLOW
    announce("small after overflow")
    out, _ = engine.run(dg, sx.SX_BFS, 0)
    np.testing.assert_array_equal(engine.to_host(dg, sx.SX_BFS, out), np.arange(40))
    dg.close()
