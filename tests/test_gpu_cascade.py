"""BFS and SSSP on sparse graphs of high diameter under the default policy
(windowed cascades) against the oracle: rows around the lengths at which the
kernel shares them (4, 16, 64 arcs; hubs of 4,096), frontiers that outgrow the
LDS queues or go back to the level phases, directed and renumbered graphs,
bucket widths from 1 up, several runs on one loaded graph, distance overflow."""
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


def _weighted(n, edges, seed, hi=1000, directed=False):
    w = np.random.default_rng(seed).integers(1, hi + 1, len(edges))
    return gen.from_edges(n, edges, w, directed=directed)


def _path(a, b):
    return [(i, i + 1) for i in range(a, b)]


def _comb(tooth_sizes, spacing=9):
    """A path with stars of the given sizes hanging off it."""
    n = spacing * (len(tooth_sizes) + 3)
    edges, at = _path(0, n - 1), n
    for k, s in enumerate(tooth_sizes):
        edges += [(spacing * (k + 2), at + j) for j in range(s)]
        at += s
    return _weighted(at, edges, 5)


def _path_blob_path(blob, degree, tail, seed):
    """path - random graph of `blob` vertices - path."""
    r = np.random.default_rng(seed)
    mid = r.integers(tail, tail + blob, (blob * degree // 2, 2))
    n = 2 * tail + blob
    edges = np.concatenate([_path(0, tail), mid, _path(tail + blob - 1, n - 1)])
    return _weighted(n, edges, seed + 1)


def _ladder(n, width, seed, directed=False):
    """Layers of `width` vertices, each joined to two of the next layer."""
    r = np.random.default_rng(seed)
    layers = n // width
    v = np.arange((layers - 1) * width)
    up = [(v, (v // width + 1) * width + r.integers(0, width, len(v))) for _ in range(2)]
    return _weighted(layers * width, np.concatenate([np.stack(e, axis=1) for e in up]), seed, directed=directed)


GRAPHS = [
    ("path-40", lambda: _weighted(40, _path(0, 39), 1)),
    ("path-5000", lambda: _weighted(5000, _path(0, 4999), 2)),
    ("grid-33", lambda: gen.grid(33, 0.1, seed=4, weights=(1, 1000))),
    ("grid-200", lambda: gen.grid(200, 0.1, seed=5, weights=(1, 1000))),
    ("comb-rows", lambda: _comb([1, 2, 3, 14, 15, 16, 61, 62, 63, 64, 300])),
    # rows of 4,095 to 4,098 arcs; then more hubs in a row than listed in LDS at once
    ("comb-hubs", lambda: _comb([4093, 4094, 4095, 4096, 5, 9000, 4094])),
    ("comb-many-hubs", lambda: _comb([4200] * 12, spacing=1)),
    # a star whose leaves start paths: the queue overflows at once
    ("broom", lambda: _weighted(60000, _path(0, 60) + [(60, 61 + i) for i in range(3000)]
                                + [(61 + i, 3061 + i) for i in range(56939)], 7)),
    ("ladder-4000", lambda: _ladder(400000, 4000, 8)),
    ("ladder-directed", lambda: _ladder(100000, 700, 9, directed=True)),
    # the frontier leaves the cascade and comes back to it
    ("path-blob-path", lambda: _path_blob_path(400000, 5, 600, 11)),
]


@pytest.mark.parametrize("name,make", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_cascade_exact(engine, name, make):
    g = make()
    assert g.m < 8 * g.n
    far = g.n - 1 if not g.directed else 0
    srcs = sorted({0, g.n // 2 if not g.directed else 1, far})
    refs = {s: (oracle.bfs_g(g, s), oracle.sssp_g(g, s)) for s in srcs}
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        for s in srcs + srcs[:1]:
            announce(f"cascade bfs {name} reorder={reorder} src={s}")
            out, st = engine.run(dg, sx.SX_BFS, s)
            np.testing.assert_array_equal(engine.to_host(dg, sx.SX_BFS, out), refs[s][0])
            assert st["iterations"] == refs[s][0].max() + 1
            for delta in (1 << 20, 4000, 300) if g.n > 10000 else (1 << 20, 4000, 300, 1):
                announce(f"cascade sssp {name} reorder={reorder} src={s} delta={delta}")
                out, _ = engine.run(dg, sx.SX_SSSP, s, sssp_delta=delta)
                np.testing.assert_array_equal(engine.to_host(dg, sx.SX_SSSP, out), refs[s][1])
        dg.close()


def test_cascade_static_and_overflow(engine):
    g = gen.grid(90, 0.1, seed=3, weights=(1, 1000))
    s = gen.max_degree_vertex(g)
    dg = engine.load(g)
    for algo, ref, kw in [(sx.SX_BFS, oracle.bfs_g(g, s), {}), (sx.SX_SSSP, oracle.sssp_g(g, s), {"sssp_delta": 900})]:
        announce(f"cascade static algo={algo}")
        out, _ = engine.run_static(dg, algo, s, **kw)
        np.testing.assert_array_equal(engine.to_host(dg, algo, out), ref)
    dg.close()
    # the sum passes 2^32 after the run has gone over to the cascade
    p = gen.from_edges(60, _path(0, 59), [1] * 30 + [1 << 28] * 29)
    dp = engine.load(p)
    announce("cascade overflow")
    with pytest.raises(sx.SxError) as ei:
        engine.run(dp, sx.SX_SSSP, 0, sssp_delta=1000)
    assert ei.value.status == sx.SX_EOVERFLOW
    announce("cascade after overflow")
    out, _ = engine.run(dp, sx.SX_BFS, 0)
    np.testing.assert_array_equal(engine.to_host(dp, sx.SX_BFS, out), np.arange(60))
    dp.close()


@pytest.mark.parametrize("team", [1, 3, 32])
def test_cascade_batch(engine, team):
    """Queries of a batch on the same graphs, by teams of 1 to 32 workgroups;
    each graph is queried several times, so workspaces carry earlier stamps."""
    import torch
    loaded, queries, outs, refs = [], [], [], []
    for name, make in GRAPHS:
        g = make()
        dg = engine.load(g)
        loaded.append(dg)
        for k, s in enumerate((0, g.n - 1 if not g.directed else 1, 0)):
            algo = sx.SX_BFS if k == 2 or (k + len(loaded)) % 2 else sx.SX_SSSP
            outs.append(torch.empty(g.n, dtype=torch.int32, device="cuda"))
            queries.append((dg.handle, algo, s, outs[-1].data_ptr()))
            refs.append((name, algo, s, oracle.bfs_g(g, s) if algo == sx.SX_BFS else oracle.sssp_g(g, s)))
    cfg = sx.sx_batch_config(team, 0, 0)
    for rep in range(2):
        announce(f"cascade batch team={team} rep {rep}")
        _, stats = sx.sx_run_batch(engine.ctx, queries, cfg=cfg, stream=engine.stream())
        for (name, algo, s, ref), out, st in zip(refs, outs, stats):
            got = out.cpu().numpy().view(ref.dtype)
            np.testing.assert_array_equal(got, ref, err_msg=f"{name} algo={algo} src={s}")
            if algo == sx.SX_BFS:
                assert st["iterations"] == ref.max() + 1
    for dg in loaded:
        dg.close()
