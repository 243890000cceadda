"""Batches by the kernel they take: dense graphs only (no cascade in it), sparse
ones among them (with it), and sparse ones under a policy that fixes a choice
(without it again); small and large teams."""
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


DENSE = [lambda: gen.rmat(12, seed=1, weights=(1, 64)), lambda: gen.random_graph(300, 0.2, seed=2, weights=(1, 9))]
SPARSE = [lambda: gen.grid(90, 0.1, seed=3, weights=(1, 1000)), lambda: gen.from_edges(3, [(0, 1)], [5])]


@pytest.mark.parametrize("team", [1, 4, 32])
@pytest.mark.parametrize("name,makes,pol", [("dense", DENSE, None), ("mixed", DENSE + SPARSE, None),
                                            ("mixed-bins", DENSE + SPARSE, sx.Policy(bin_small=32))])
def test_batch_kernels(engine, name, makes, pol, team):
    import torch
    loaded, queries, outs, refs = [], [], [], []
    for make in makes:
        g = make()
        dg = engine.load(g)
        loaded.append(dg)
        for algo, fn in ((sx.SX_BFS, oracle.bfs_g), (sx.SX_SSSP, oracle.sssp_g)):
            for s in (0, g.n - 1):
                outs.append(torch.empty(g.n, dtype=torch.int32, device="cuda"))
                queries.append((dg.handle, algo, s, outs[-1].data_ptr()))
                refs.append(fn(g, s))
    announce(f"batch kernels {name} team={team}")
    sx.sx_run_batch(engine.ctx, queries, pol=pol.c() if pol else None, cfg=sx.sx_batch_config(team, 0, 0),
                    stream=engine.stream())
    for k, (ref, out) in enumerate(zip(refs, outs)):
        np.testing.assert_array_equal(out.cpu().numpy().view(ref.dtype), ref, err_msg=f"query {k}")
    for dg in loaded:
        dg.close()
