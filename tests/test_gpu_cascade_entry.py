"""Which runs on sparse graphs beyond the one-workgroup size (24,576 vertices)
go over to the cascade: seen by launches far below the levels, with results equal
to the oracle's.  BFS under the heuristic and the learned policy (its network is
asked about heavy frontiers only) and without allocation, SSSP with buckets; not
SSSP without them, whose automatic width on a graph this small is none."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from oracle import mlp as ref
from paper_1812_04070_amd import gen
from tests.gpu_util import announce, run

pytestmark = pytest.mark.gpu

LEARNED = sx.Policy(policy=sx.SX_POLICY_LEARNED)


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    sx.sx_policy_load_mlp(e.ctx, np.zeros_like(ref.init_params(1), dtype=np.float32))
    yield e
    e.close()


@pytest.fixture(scope="module")
def grid():
    g = gen.grid(200, 0.1, seed=11, weights=(1, 1000))
    s = gen.max_degree_vertex(g)
    return g, s, oracle.bfs_g(g, s), oracle.sssp_g(g, s)


@pytest.mark.parametrize("pol", [None, LEARNED], ids=["heuristic", "learned"])
@pytest.mark.parametrize("reorder", [False, True])
def test_enters(engine, grid, pol, reorder):
    g, s, depth, dist = grid
    levels = int(depth.max()) + 1
    dg = engine.load(g, reorder=reorder)
    for rep in range(2):
        announce(f"cascade entry reorder={reorder} {pol} rep {rep}")
        out, st = run(engine, g, sx.SX_BFS, s, pol, dg=dg)
        np.testing.assert_array_equal(out, depth)
        assert st["iterations"] == levels and st["launches"] < levels / 3
        out, st = run(engine, g, sx.SX_SSSP, s, pol, dg=dg, sssp_delta=4000)
        np.testing.assert_array_equal(out, dist)
        assert st["launches"] < levels / 3
    dg.close()


def test_enters_without_allocation(engine, grid):
    g, s, depth, dist = grid
    dg = engine.load(g)
    for algo, expect, kw in ((sx.SX_BFS, depth, {}), (sx.SX_SSSP, dist, {"sssp_delta": 4000})):
        announce(f"cascade entry static algo={algo}")
        out, st = engine.run_static(dg, algo, s, **kw)
        np.testing.assert_array_equal(engine.to_host(dg, algo, out), expect)
        assert 1 < st["launches"] < (int(depth.max()) + 1) / 3
    dg.close()


def test_automatic_width_of_a_small_graph_is_none(engine, grid):
    g, s, depth, dist = grid
    dg = engine.load(g)
    stats = []
    for delta in (0, sx.SX_DELTA_AUTO):
        announce(f"cascade entry sssp delta={delta}")
        out, st = run(engine, g, sx.SX_SSSP, s, None, dg=dg, sssp_delta=delta)
        np.testing.assert_array_equal(out, dist)
        stats.append(st)
        # the phases: a launch an iteration, at least one a hop
        assert st["launches"] >= st["iterations"] >= int(depth.max())
    dg.close()
    assert stats[0]["iterations"] == pytest.approx(stats[1]["iterations"], abs=3)
