"""SSSP on graphs without arcs in every arrangement: the source is at distance
0, every other vertex unreached, and the run ends (a sequenced run whose lists
are empty has to reach the decision that ends it)."""
from __future__ import annotations

import numpy as np
import pytest

import paper_1812_04070_amd as sx
from paper_1812_04070_amd import gen
from tests.gpu_util import ARMS, announce, run

pytestmark = pytest.mark.gpu

EXTRA = [("push-seq", sx.Policy(direction=sx.SX_DIR_PUSH, fused=sx.SX_SEQUENCED)),
         ("online-seq", sx.Policy(filter=sx.SX_FILTER_ONLINE, fused=sx.SX_SEQUENCED))]


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


def _check(engine, n, arms):
    g = gen.from_edges(n, [], [])
    for reorder in (False, True):
        dg = engine.load(g, reorder=reorder)
        for src in sorted({0, n // 2, n - 1}):
            ref = np.full(n, 0xFFFFFFFF, dtype=np.uint32)
            ref[src] = 0
            for name, pol in arms:
                for delta in (0, sx.SX_DELTA_AUTO, 5):
                    announce(f"edgeless sssp n={n} reorder={reorder} src={src} {name} delta={delta}")
                    out, _ = run(engine, g, sx.SX_SSSP, src, pol, dg=dg, sssp_delta=delta)
                    np.testing.assert_array_equal(out, ref)
        dg.close()


@pytest.mark.parametrize("n", [1, 2, 100])
def test_edgeless_small(engine, n):
    _check(engine, n, ARMS + EXTRA)


def test_edgeless_past_the_one_workgroup_path(engine):
    _check(engine, 24577, ARMS[:1])
