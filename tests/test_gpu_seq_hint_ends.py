"""Runs of the sequenced arrangement asked for by name (neither the
one-workgroup kernel nor the cascade takes them) whose first batch of launches
is too short, too long or just right, also on a renumbered graph, whose result
is mapped behind the first batch when that batch is expected to end the run
and again when it did not."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from paper_1812_04070_amd import gen
from tests.gpu_util import announce, run

pytestmark = pytest.mark.gpu

SEQ = sx.Policy(fused=sx.SX_SEQUENCED)


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


@pytest.mark.parametrize("reorder", [False, True])
def test_hint_too_low_and_too_high_sequenced(engine, reorder):
    n = 1500
    g = gen.from_edges(n, [(i, i + 1) for i in range(n - 1)], [1 + (i % 7) for i in range(n - 1)])
    dg = engine.load(g, reorder=reorder)
    for algo, oracle_fn in [(sx.SX_BFS, oracle.bfs_g), (sx.SX_SSSP, oracle.sssp_g), (sx.SX_WCC, None)]:
        for src in (n // 2, 0, n // 2, n - 1):
            announce(f"seq hint path-{n} algo={algo} src={src} reorder={reorder}")
            out, st = run(engine, g, algo, src, SEQ, dg=dg)
            ref = oracle_fn(g, src) if oracle_fn else np.zeros(n, dtype=np.int32)
            np.testing.assert_array_equal(out, ref)
            # a launch per hop: no other path took the run
            assert algo == sx.SX_WCC or st["launches"] >= max(src, n - 1 - src)
    dg.close()


@pytest.mark.parametrize("reorder", [False, True])
def test_near_run_after_far_run_and_back(engine, reorder):
    """A near run sets a hint below what the far one needs and is then what
    the far one's hint is too long for."""
    g = gen.rmat(14, seed=8, weights=(1, 64))
    tail = g.n + np.arange(40)
    src, dst = np.repeat(np.arange(g.n), np.diff(g.offsets)), g.indices
    edges = np.concatenate([np.stack([src, dst], axis=1),
                            np.stack([np.concatenate([[gen.max_degree_vertex(g)], tail[:-1]]), tail], axis=1)])
    h = gen.from_edges(g.n + 40, edges, 1 + np.arange(len(edges)) % 9)
    iso = int(np.flatnonzero(h.out_degree() == 0)[0])
    dg = engine.load(h, reorder=reorder)
    for algo, oracle_fn in [(sx.SX_BFS, oracle.bfs_g), (sx.SX_SSSP, oracle.sssp_g)]:
        for s in (iso, gen.max_degree_vertex(g), int(tail[-1]), iso, int(tail[-1])):
            announce(f"seq hint rmat-tail algo={algo} src={s} reorder={reorder}")
            out, _ = run(engine, h, algo, s, SEQ, dg=dg)
            np.testing.assert_array_equal(out, oracle_fn(h, s))
    dg.close()


def test_repeated_cascade_run_enqueues_what_it_needs(engine):
    """Runs that the cascade takes on near their end: the launches before it and
    those from it on are sized by the last run's, so that a repeated run
    enqueues about as many as the phases alone do (the margin of two once more,
    the step that finds the list empty, and a few for windows cut short)."""
    r = np.random.default_rng(3)
    n = 1 << 21
    g = gen.from_edges(n, r.integers(0, n, (2 * n, 2)), r.integers(1, 65, 2 * n))
    s = gen.max_degree_vertex(g)
    ref = oracle.bfs_g(g, s)
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        launches = {}
        for name, pol in (("phases", SEQ), ("cascade", None)):
            for rep in range(4):
                announce(f"cascade tail {name} reorder={reorder} rep {rep}")
                out, st = run(engine, g, sx.SX_BFS, s, pol, dg=dg)
                np.testing.assert_array_equal(out, ref)
                launches[name, rep] = st["launches"]
        print(f"[seq-hint] cascade tail launches {launches}", flush=True)
        assert all(launches["cascade", k] <= launches["phases", 3] + 8 for k in (1, 2, 3)), launches
        dg.close()
