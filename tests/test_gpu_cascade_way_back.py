"""Cascades that meet a part of the graph of low diameter and go back to the
level phases (lists of more than 2^16 vertices), some of them several times in
a run: BFS depths and level counts, SSSP distances, alone and in a batch,
directed and renumbered, and the work of a BFS, which the way back bounds."""
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


def _chain(parts, seed, directed=False):
    """Paths (an int: its vertices) and random graphs (vertices, degree) in a row."""
    r = np.random.default_rng(seed)
    edges, at = [], 0
    for p in parts:
        size = p if isinstance(p, int) else p[0]
        if isinstance(p, int):
            v = np.arange(at, at + size - 1)
            edges.append(np.stack([v, v + 1], axis=1))
        else:
            edges.append(r.integers(at, at + size, (size * p[1] // 2, 2)))
        if at:
            edges.append(np.array([[at - 1, at]]))
        at += size
    edges = np.concatenate(edges)
    return gen.from_edges(at, edges, r.integers(1, 1001, len(edges)), directed=directed)


GRAPHS = [
    ("short-path-blob", lambda: _chain([20, (400000, 6)], 1)),
    ("path-blob-path", lambda: _chain([600, (400000, 5), 600], 2)),
    ("three-blobs", lambda: _chain([50, (250000, 6), 90, (300000, 7), 40, (250000, 4), 60], 3)),
    ("directed", lambda: _chain([60, (600000, 14), 60], 4, directed=True)),
    # a frontier of 70,000 vertices without out-arcs: few arcs, a long list
    ("sinks", lambda: gen.from_edges(70100, [(i, i + 1) for i in range(29)] + [(29, 30 + i) for i in range(70000)],
                                     1 + np.arange(70029) % 9, directed=True)),
]


@pytest.mark.parametrize("name,make", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_way_back_exact(engine, name, make):
    g = make()
    assert g.m < 8 * g.n
    srcs = (0, g.n - 1) if not g.directed else (0, 3)
    refs = {s: (oracle.bfs_g(g, s), oracle.sssp_g(g, s)) for s in srcs}
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        for s in srcs + srcs[:1]:
            announce(f"way back bfs {name} reorder={reorder} src={s}")
            out, st = engine.run(dg, sx.SX_BFS, s)
            np.testing.assert_array_equal(engine.to_host(dg, sx.SX_BFS, out), refs[s][0])
            assert st["iterations"] == refs[s][0].max() + 1
            for delta in (1 << 20, 4000, 300):
                announce(f"way back sssp {name} reorder={reorder} src={s} delta={delta}")
                out, _ = engine.run(dg, sx.SX_SSSP, s, sssp_delta=delta)
                np.testing.assert_array_equal(engine.to_host(dg, sx.SX_SSSP, out), refs[s][1])
        dg.close()


def test_way_back_bounds_the_work(engine):
    """Every arc once in the phases, and fewer than all of them again in the
    steps before the list is seen to be long: it then holds 2^16 of the blob's
    400,000 vertices."""
    g = _chain([600, (400000, 5), 600], 2)
    dg = engine.load(g)
    for s in (0, g.n - 1):
        announce(f"way back work src={s}")
        _, st = engine.run(dg, sx.SX_BFS, s)
        assert st["edges_inspected"] <= 2 * g.m
    dg.close()


@pytest.mark.parametrize("team", [3, 32])
def test_way_back_batch(engine, team):
    import torch
    loaded, queries, outs, refs = [], [], [], []
    for name, make in GRAPHS:
        g = make()
        dg = engine.load(g)
        loaded.append(dg)
        for k, s in enumerate((0, g.n - 1 if not g.directed else 1, 0, 2)):
            algo = sx.SX_BFS if k % 2 == 0 else sx.SX_SSSP
            outs.append(torch.empty(g.n, dtype=torch.int32, device="cuda"))
            queries.append((dg.handle, algo, s, outs[-1].data_ptr()))
            refs.append((name, algo, s, oracle.bfs_g(g, s) if algo == sx.SX_BFS else oracle.sssp_g(g, s)))
    cfg = sx.sx_batch_config(team, 0, 0)
    for rep in range(2):
        announce(f"way back batch team={team} rep {rep}")
        _, stats = sx.sx_run_batch(engine.ctx, queries, cfg=cfg, stream=engine.stream())
        for (name, algo, s, ref), out, st in zip(refs, outs, stats):
            np.testing.assert_array_equal(out.cpu().numpy().view(ref.dtype), ref, err_msg=f"{name} algo={algo} src={s}")
            if algo == sx.SX_BFS:
                assert st["iterations"] == ref.max() + 1
    for dg in loaded:
        dg.close()
