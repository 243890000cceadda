"""SSSP steps that hold a quarter of the arcs and more on graphs of 6 M arcs and
more: their improved vertices are listed by a scan.  Whole-number distances,
equal to the oracle's: R-MAT graphs both sides of the size, directed,
renumbered, a dense random graph whose every step is heavy, buckets of the
caller's, repeated runs, and a sum past 32 bits in such a step."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from paper_1812_04070_amd import gen
from tests.gpu_util import announce, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


def _dense(n, m, seed, lo, hi, directed=False):
    r = np.random.default_rng(seed)
    e = r.integers(0, n, (m, 2))
    e = np.unique(e[e[:, 0] < e[:, 1]] if not directed else e[e[:, 0] != e[:, 1]], axis=0)
    return gen.from_edges(n, e, r.integers(lo, hi + 1, len(e)), directed=directed)


def _check(engine, g, sources, **kw):
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        for s in sources:
            ref = oracle.sssp_g(g, s)
            for _ in range(2):
                out, _ = run(engine, g, sx.SX_SSSP, s, dg=dg, **kw)
                np.testing.assert_array_equal(out, ref)
        dg.close()


@pytest.mark.parametrize("scale,directed", [(17, False), (18, False), (18, True), (19, True)])
def test_sssp_rmat(engine, scale, directed):
    announce(f"sssp heavy rmat {scale} directed {directed}")
    g = gen.rmat(scale, seed=scale, directed=directed, weights=(1, 64))
    deg = g.out_degree()
    _check(engine, g, [int(deg.argmax()), int(np.flatnonzero(deg == 1)[0])])


@pytest.mark.parametrize("delta", [0, 1000])
def test_sssp_dense(engine, delta):
    """Every step from the second on is heavy; buckets of the caller's are
    not marked."""
    announce(f"sssp heavy dense delta {delta}")
    _check(engine, _dense(6000, 7_500_000, 3, 1, 100_000), [0], sssp_delta=delta)


def test_sssp_heavy_overflow(engine):
    """Distances 1.5 and 3 x 2^30 in light steps, 4.5 x 2^30 in a heavy one."""
    g = _dense(20000, 8_000_000, 5, 3 << 29, 3 << 29)
    dg = engine.load(g)
    announce("sssp heavy overflow")
    with pytest.raises(sx.SxError) as ei:
        engine.run(dg, sx.SX_SSSP, 0)
    assert ei.value.status == sx.SX_EOVERFLOW
    announce("bfs after overflow")
    out, _ = engine.run(dg, sx.SX_BFS, 0)
    np.testing.assert_array_equal(engine.to_host(dg, sx.SX_BFS, out), oracle.bfs_g(g, 0))
    dg.close()
