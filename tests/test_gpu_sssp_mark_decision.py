"""What an SSSP step that only marks its improvements leaves to the rest of the
run: the end is seen and counted as without marking, and a later decision of
the learned policy is given the same features (frontier before, vertices
reached so far).  The reference is the sequenced arrangement asked for by
name, which lists every step's improvements online; unit weights make the
frontiers the same in both."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from oracle import mlp as ref
from paper_1812_04070_amd import gen
from tests.gpu_util import announce, run

pytestmark = pytest.mark.gpu

MARK_ARCS = 6_000_000   # graphs of fewer arcs list online


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


def _unit(n, edges):
    return gen.from_edges(n, edges, np.ones(len(edges), dtype=np.int64))


def test_marked_step_that_improves_nothing_ends_the_run(engine):
    n = 2500
    g = _unit(n, np.stack(np.triu_indices(n, 1), axis=1))
    assert g.m >= MARK_ARCS
    dg = engine.load(g)
    for pol in (None, sx.Policy(fused=sx.SX_SEQUENCED)):
        announce(f"complete graph sssp {pol}")
        out, st = run(engine, g, sx.SX_SSSP, 7, pol, dg=dg)
        np.testing.assert_array_equal(out, np.arange(n) != 7)
        assert st["iterations"] == 2
    dg.close()


def test_features_after_marked_steps(engine):
    """Layers of which the first two steps hold over a quarter of the arcs each
    and are marked, the later ones (over 2^18 arcs) are decided upon."""
    r = np.random.default_rng(4)
    sizes = [1, 2000, 2000] + [1000] * 5
    first = np.concatenate([[0], np.cumsum(sizes)])
    v = np.arange(2000)
    edges = [np.stack([np.zeros(2000, dtype=np.int64), 1 + v], axis=1),
             np.stack([np.repeat(1 + v, 2000), np.tile(2001 + v, 2000)], axis=1)]
    for k in range(2, len(sizes) - 1):
        edges.append(np.stack([r.integers(first[k], first[k + 1], 200_000),
                               r.integers(first[k + 1], first[k + 2], 200_000)], axis=1))
    g = _unit(int(first[-1]), np.concatenate(edges))
    assert g.m >= MARK_ARCS
    # a network without a preference: every choice stays the rule's
    sx.sx_policy_load_mlp(engine.ctx, np.zeros_like(ref.init_params(1), dtype=np.float32))
    dg = engine.load(g)
    dist, seen = oracle.sssp_g(g, 0), []
    for fused in (sx.SX_SEQUENCED, sx.SX_FUSE_AUTO):
        announce(f"layers sssp learned fused={fused}")
        out, st = run(engine, g, sx.SX_SSSP, 0, sx.Policy(policy=sx.SX_POLICY_LEARNED, fused=fused), dg=dg)
        np.testing.assert_array_equal(out, dist)
        assert st["policy_evals"] > 0
        seen.append((st["iterations"], list(st["policy_x"])))
    dg.close()
    assert seen[0] == seen[1]
