"""A run that fails on a renumbered graph leaves the caller's array as it was:
the array handed to an SSSP whose distances pass 32 bits, in the one-workgroup
kernel and in a sequenced run whose first batch was expected to end it (the
mapping into the array is then enqueued before the host knows how the run
ended), and belief propagation's priors after an invalid one."""
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


@pytest.mark.parametrize("bad", [0.0, 1.0, float("nan")])
def test_invalid_prior_keeps_the_priors(engine, bad):
    import torch
    g = gen.rmat(10, seed=5, weights=(1, 64))
    prior = gen.bp_priors(g.n, seed=3)
    prior[g.n // 3] = bad
    dg = engine.load(g, reorder=True)
    out = torch.from_numpy(prior.copy()).to(engine.device)
    for iters in (1, 6):
        announce(f"bp prior {bad} iters={iters} reordered")
        with pytest.raises(sx.SxError) as ei:
            engine.run(dg, sx.SX_BP, out=out, bp_iters=iters)
        assert ei.value.status == sx.SX_EINVAL
        np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), prior.view(np.uint32))
    dg.close()


@pytest.mark.parametrize("fused", [sx.SX_FUSE_AUTO, sx.SX_SEQUENCED])
def test_sssp_overflow_keeps_the_array(engine, fused):
    import torch
    # two paths; the second one's sums pass 2^32 with its third vertex
    edges = [(i, i + 1) for i in range(19)] + [(i, i + 1) for i in range(20, 39)]
    g = gen.from_edges(40, edges, [1] * 19 + [1 << 31] * 19)
    pol = sx.Policy(fused=fused)
    dg = engine.load(g, reorder=True)
    for rep in range(2):
        announce(f"overflow reordered fused={fused} rep {rep}: the near path")
        out, _ = engine.run(dg, sx.SX_SSSP, 0, pol)
        np.testing.assert_array_equal(engine.to_host(dg, sx.SX_SSSP, out), oracle.sssp_g(g, 0))
        out = torch.full((g.n,), 77, dtype=torch.int32, device=engine.device)
        announce(f"overflow reordered fused={fused} rep {rep}: the far path")
        with pytest.raises(sx.SxError) as ei:
            engine.run(dg, sx.SX_SSSP, 20, pol, out=out)
        assert ei.value.status == sx.SX_EOVERFLOW
        assert bool((out == 77).all())
    dg.close()
