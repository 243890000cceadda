"""PageRank and belief propagation on sparse graphs either side of the rule that
says whether a workgroup copies the first vertices' values into its LDS: by the
default grid it does not, on 8 workgroups it does, and the sums, whose order does
not depend on the grid, have the same bits (no vertex without out-arcs, so no
partial sums per workgroup are used); against the FP64 oracle within the bounds
of the other PageRank (relative L1 1e-6) and belief-propagation (1e-5) tests."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from paper_1812_04070_amd import gen
from tests.gpu_util import announce, rel_l1

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


@pytest.mark.parametrize("side", [200, 240, 300, 420])
def test_same_bits_with_and_without_the_copy(engine, side):
    g = gen.grid(side, 0.0, seed=2, weights=(1, 64))
    assert g.out_degree().min() > 0
    prior = gen.bp_priors(g.n, seed=side)
    dg = engine.load(g)
    ranks, beliefs = [], []
    for pol in (None, sx.Policy(grid_wgs=8), sx.Policy(grid_wgs=100)):
        announce(f"hot sources grid-{side} {pol}")
        out, _ = engine.run(dg, sx.SX_PAGERANK, -1, pol, pr_iters=12)
        ranks.append(engine.to_host(dg, sx.SX_PAGERANK, out).copy())
        out, _ = engine.run(dg, sx.SX_BP, -1, pol, prior=prior, bp_kappa=0.6, bp_iters=6)
        beliefs.append(engine.to_host(dg, sx.SX_BP, out).copy())
    dg.close()
    for a in (ranks, beliefs):
        for x in a[1:]:
            np.testing.assert_array_equal(x.view(np.uint32), a[0].view(np.uint32))
    assert rel_l1(ranks[0], oracle.pagerank_g(g, iters=12)) <= 1e-6
    assert rel_l1(beliefs[0], oracle.bp_g(g, prior.astype(np.float64), 0.6, 6)) <= 1e-5
