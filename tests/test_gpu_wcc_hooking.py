"""Connected components by hooking (the default policy) against the oracle's
union-find, at the sizes where its kernels change course: vertex counts around
the wavefront and the workgroup, rows around the lengths a wavefront and a
workgroup share, components besides the largest one (whose rows are skipped),
long parent chains; renumbered graphs and the no-allocation call too."""
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


def _stars(*sizes):
    """Disjoint stars, centres last within each, sparse ids first."""
    edges, at = [], 0
    for s in sizes:
        edges += [(at + i, at + s) for i in range(s)]
        at += s + 1
    return gen.from_edges(at, edges)


def _shuffled_paths(n, k, seed):
    """k interleaved paths over a random order of n vertices."""
    p = np.random.default_rng(seed).permutation(n)
    return gen.from_edges(n, np.stack([p[:-k], p[k:]], axis=1))


GRAPHS = [
    *[(f"path-{n}", lambda n=n: gen.from_edges(n, [(i, i + 1) for i in range(n - 1)]))
      for n in (2, 63, 64, 65, 511, 512, 513, 1025)],
    ("path-300000", lambda: gen.from_edges(300000, np.stack([np.arange(299999), np.arange(1, 300000)], axis=1))),
    ("shuffled-paths", lambda: _shuffled_paths(100003, 7, 5)),
    # rows of 2 + 31/32/33 and 2 + 1023/1024/1025 arcs beside a larger component
    ("stars-wave", lambda: _stars(5000, 33, 34, 35, 1, 2, 3)),
    ("stars-group", lambda: _stars(20000, 1025, 1026, 1027, 64)),
    ("equal-halves", lambda: _stars(3000, 3000)),
    ("random-many-components", lambda: gen.from_edges(50000, np.random.default_rng(3).integers(0, 50000, (26000, 2)))),
    ("grid-300-holes", lambda: gen.grid(300, 0.45, seed=7)),
    ("grid-301", lambda: gen.grid(301, 0.1, seed=8)),
    ("rmat17-sparse", lambda: gen.rmat(17, edge_factor=2, seed=9)),
    ("edgeless-700", lambda: gen.from_edges(700, [])),
]


@pytest.mark.parametrize("name,make", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_labels(engine, name, make):
    g = make()
    ref = oracle.wcc_g(g)
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        for rep in range(3):
            announce(f"wcc hooking {name} reorder={reorder} rep {rep}")
            out, st = engine.run(dg, sx.SX_WCC)
            np.testing.assert_array_equal(engine.to_host(dg, sx.SX_WCC, out), ref)
            assert st["launches"] == (7 if reorder else 6)
        if not reorder:
            announce(f"wcc hooking {name} static")
            out, _ = engine.run_static(dg, sx.SX_WCC)
            np.testing.assert_array_equal(engine.to_host(dg, sx.SX_WCC, out), ref)
        dg.close()
