"""Connected components at the most arcs a graph may have (2^31 - 2), where the
last rows end within a step of the largest int32: a large component in front,
pairs joined by 1,023 parallel edges whose rows a wavefront walks, the last of
them ending at the limit, and isolated vertices behind it."""
from __future__ import annotations

import numpy as np
import pytest

import paper_1812_04070_amd as sx
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu

N, D, PAIRS, R, ALONE = 21483, 99960, 21, 1023, 3
ARCS = N * D + PAIRS * 2 * R


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < (100 << 30):
        pytest.skip("needs 100 GB of device memory")
    e = sx.Engine(0)
    yield e
    e.close()


def test_wcc_at_the_arc_limit(engine):
    import torch
    assert ARCS == 2**31 - 2
    n = N + 2 * PAIRS + ALONE
    idx = torch.empty(ARCS, dtype=torch.int32, device="cuda")
    # vertex v of the large component leads to v +- 1 .. v +- D / 2 around a ring
    # of N (several times over: a multigraph)
    step = torch.arange(1, D // 2 + 1, device="cuda", dtype=torch.int32)
    step = torch.cat([step, -step])
    for v0 in range(0, N, 400):
        v = torch.arange(v0, min(v0 + 400, N), device="cuda", dtype=torch.int32)
        idx[v0 * D:(v0 + len(v)) * D] = torch.remainder(v[:, None] + step[None, :], N).reshape(-1)
    a = N + 2 * torch.arange(PAIRS, device="cuda", dtype=torch.int32)
    idx[N * D:] = torch.stack([a + 1, a], dim=1).repeat_interleave(R, dim=1).reshape(-1)
    counts = np.array([D] * N + [R] * (2 * PAIRS) + [0] * ALONE, dtype=np.int64)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda()
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    announce(f"wcc n={n} m={ARCS}")
    g = sx.sx_graph_load(engine.ctx, sx.sx_graph_desc(n, ARCS, off.data_ptr(), idx.data_ptr(), None, None, None, None,
                                                      sx.SX_DEVICE_PTRS | sx.SX_UNDIRECTED), engine.stream())
    p = sx.sx_program_register(engine.ctx, sx.SX_WCC)
    try:
        sx.sx_run(p, g, -1, out.data_ptr(), engine.stream())
        ref = np.concatenate([np.zeros(N, dtype=np.int64), np.repeat(N + 2 * np.arange(PAIRS), 2),
                              N + 2 * PAIRS + np.arange(ALONE)])
        np.testing.assert_array_equal(out.cpu().numpy(), ref)
    finally:
        sx.sx_program_destroy(p)
        sx.sx_graph_destroy(g)
