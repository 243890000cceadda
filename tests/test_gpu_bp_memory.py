"""Belief propagation where the device has little memory left: the couplings are
not stored (an array of 4 bytes an arc, at most an eighth of what is free), what
is free stays free, and the beliefs have the bits of a run that stores them."""
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


def test_bp_without_room_for_the_couplings(engine):
    import torch
    g = gen.rmat(20, seed=6, weights=(1, 64))
    prior = gen.bp_priors(g.n, seed=7)
    dg = engine.load(g)
    p = torch.from_numpy(prior).to(engine.device)
    outs = [torch.empty(g.n, dtype=torch.float32, device=engine.device) for _ in range(3)]
    held = []
    try:
        # what is left: less than 8 times the array, more than the array itself
        room = 6 * 4 * g.m
        torch.cuda.empty_cache()
        try:
            while torch.cuda.mem_get_info()[0] > room + (64 << 20):
                held.append(torch.empty(min(16 << 30, torch.cuda.mem_get_info()[0] - room), dtype=torch.uint8,
                                        device=engine.device))
        except torch.cuda.OutOfMemoryError:
            pytest.skip("the device's memory is not ours to fill")
        free = torch.cuda.mem_get_info()[0]
        assert 4 * g.m < free < 8 * 4 * g.m
        for rep in range(2):
            announce(f"bp with {free >> 20} MiB free, rep {rep}")
            engine.run(dg, sx.SX_BP, -1, prior=p, out=outs[rep], bp_kappa=0.6, bp_iters=5)
            assert torch.cuda.mem_get_info()[0] >= free - (8 << 20)
    finally:
        held.clear()
        torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    announce("bp with room")
    engine.run(dg, sx.SX_BP, -1, prior=p, out=outs[2], bp_kappa=0.6, bp_iters=5)
    assert torch.cuda.mem_get_info()[0] <= free - 4 * g.m + (8 << 20)
    got = [o.cpu().numpy() for o in outs]
    dg.close()
    for x in got[1:]:
        np.testing.assert_array_equal(x.view(np.uint32), got[0].view(np.uint32))
    # the bound of the other belief-propagation tests
    assert rel_l1(got[0], oracle.bp_g(g, prior.astype(np.float64), 0.6, 5)) <= 1e-5
