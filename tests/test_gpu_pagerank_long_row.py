"""PageRank of a vertex whose row one workgroup walks with the next ids in flight
(more than 32,768 arcs), and of the rows just below: lengths around that limit,
around a round of 4,096 arcs and around the workgroup's 1,024 threads, fixed
iterations and to a tolerance.  Against the FP64 oracle: relative L1 1e-6 as in
the other PageRank tests, pr_tol + 3e-6 to a tolerance."""
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


@pytest.mark.parametrize("arcs", [32767, 32768, 32769, 36863, 36864, 36865, 36865 + 1024, 40960 + 3 * 1024 - 1, 200001])
def test_long_row(engine, arcs):
    """`arcs` sources lead to vertex 0; the second half of them also to vertex 1,
    and every tenth has no other way out."""
    src = 2 + np.arange(arcs)
    half = src[arcs // 2:]
    edges = np.concatenate([np.stack([src, np.zeros_like(src)], axis=1), np.stack([half, np.ones_like(half)], axis=1),
                            np.stack([src[src % 10 != 0], 2 + (src[src % 10 != 0] * 7919) % arcs], axis=1)])
    g = gen.from_edges(arcs + 2, edges, directed=True)
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        announce(f"long row {arcs} reorder={reorder}")
        out, _ = engine.run(dg, sx.SX_PAGERANK, -1, pr_iters=10)
        assert rel_l1(engine.to_host(dg, sx.SX_PAGERANK, out), oracle.pagerank_g(g, iters=10)) <= 1e-6
        out, _ = engine.run(dg, sx.SX_PAGERANK, -1, pr_tol=1e-5)
        ref, _ = oracle.pagerank_fixpoint_g(g, tol=1e-15)
        got = engine.to_host(dg, sx.SX_PAGERANK, out).astype(np.float64)
        assert np.abs(got - ref).sum() <= 1e-5 + 3e-6
        dg.close()
