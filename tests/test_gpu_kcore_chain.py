"""k-core chains: vertices whose rows have exactly the lengths at which a push
step stops deleting them by itself (256 and 1,024 arcs), each taken to its level
by the deletion of the one before, hung on a clique of higher core number, with
the one-workgroup tail and without; and stars around hubs, whose decrements are
summed.  Core numbers are whole numbers: equal to the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1812_04070_amd as sx
from paper_1812_04070_amd import gen
from tests.gpu_util import announce, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def engine():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    e = sx.Engine(0)
    yield e
    e.close()


def _chains(d, chains, length, seed):
    """Chain vertices of degree d (its first: d - 1) on a clique of d + 8."""
    r = np.random.default_rng(seed)
    c = d + 8
    e = [np.stack(np.triu_indices(c, 1), axis=1)]
    for k in range(chains):
        first = c + k * length
        for i in range(length):
            v = first + i
            along = [v - 1] * (i > 0) + [v + 1] * (i + 1 < length)
            rest = d - len(along) - (i == 0)
            to = r.choice(c, rest, replace=False)
            e.append(np.stack([np.full(rest, v), to], axis=1))
            if i + 1 < length:
                e.append(np.array([[v, v + 1]]))
    return gen.from_edges(c + chains * length, np.concatenate(e).astype(np.int64), None, directed=False)


@pytest.mark.parametrize("tail", [0, -1])
@pytest.mark.parametrize("d", [255, 256, 257, 1023, 1024, 1025])
def test_kcore_chain(engine, d, tail):
    announce(f"kcore chains of degree {d} tail {tail}")
    g = _chains(d, 3, 40, seed=d)
    out, _ = run(engine, g, sx.SX_KCORE, -1, sx.Policy(kcore_tail=tail))
    np.testing.assert_array_equal(out, oracle.kcore_g(g))


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("leaves", [60000, 70000])
def test_kcore_hubs(engine, leaves, directed):
    """Steps on both sides of 65,536 arcs whose targets are a few hubs."""
    announce(f"kcore hubs leaves {leaves} directed {directed}")
    r = np.random.default_rng(leaves)
    h = 40
    ends = r.integers(0, h, (leaves, 2))
    leaf = np.arange(h, h + leaves)
    e = np.concatenate([np.stack([leaf, ends[:, 0]], axis=1), np.stack([leaf[::3], ends[::3, 1]], axis=1),
                        np.stack(np.triu_indices(h, 1), axis=1)])
    g = gen.from_edges(h + leaves, np.unique(e, axis=0), None, directed=directed)
    out, _ = run(engine, g, sx.SX_KCORE, -1, sx.Policy(kcore_tail=-1))
    np.testing.assert_array_equal(out, oracle.kcore_g(g))
