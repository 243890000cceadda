"""A caller's bucket width beyond 8 mean weights does not widen a cascade's
window: the same distances, and about the arcs of a width of 8 mean weights
(within a factor of two: the mean is sampled, the order of updates is free)."""
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


@pytest.mark.parametrize("side,lo,hi", [(700, 1, 1000), (400, 7, 7), (300, 1 << 20, 1 << 21)])
def test_wide_bucket_width(engine, side, lo, hi):
    g = gen.grid(side, 0.1, seed=5, weights=(lo, hi))
    s = gen.max_degree_vertex(g)
    ref = oracle.sssp_g(g, s)
    dg = engine.load(g)
    arcs = {}
    for delta in (4 * (lo + hi), 1 << 20, 1 << 28, (1 << 31) + 5, 0xFFFFFFFE):
        announce(f"window grid-{side} weights {lo}..{hi} delta={delta}")
        out, st = engine.run(dg, sx.SX_SSSP, s, sssp_delta=delta)
        np.testing.assert_array_equal(engine.to_host(dg, sx.SX_SSSP, out), ref)
        arcs[delta] = st["edges_inspected"]
    dg.close()
    most = 2 * arcs[4 * (lo + hi)]
    assert all(a <= most for a in arcs.values()), arcs
