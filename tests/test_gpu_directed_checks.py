"""Directed input checks that rest on one search per pair of opposite slots:
a slot without its opposite or with the wrong direction is refused whichever
end it sits at (hub or leaf, equal degrees), also with an odd number of slots;
and classes of one to many edges for the class sums, against the oracle."""

import numpy as np
import pytest

from gpu_util import device
from test_gpu_directed import check
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


def _base():
    # a hub of 40, a ring (equal degrees) and a few leaves
    n = 60
    u = np.concatenate([np.zeros(40, dtype=np.int64), np.arange(1, 40), [50]])
    v = np.concatenate([np.arange(1, 41), np.arange(2, 41), [51]])
    rp, col = G.csr_from_edges(n, u, v)
    g = G.Graph(rp, col, (np.arange(n) % 3).astype(np.uint8), 3, "checks")
    return g, G.orient(g, 0.3, 1)


def _refused(rp, col, dirs, ty, code=2):
    import torch

    import paper_2010_14058_amd as P

    dev = device()
    with pytest.raises(P.TGError) as e:
        P.count_directed(*(torch.from_numpy(np.ascontiguousarray(a)).to(dev)
                           for a in (rp, col, dirs, ty)), 3)
    assert e.value.code == code


def _slot(g, u, x):
    b, e = int(g.row_ptr[u]), int(g.row_ptr[u + 1])
    return b + int(np.searchsorted(g.col[b:e], x))


# hub side, leaf side, both sides of an edge of equal degrees, an isolated edge
SLOTS = [(0, 40), (40, 0), (10, 11), (11, 10), (50, 51), (51, 50)]


@pytest.mark.parametrize("u,x", SLOTS)
def test_one_sided_edges(u, x):
    g, dirs = _base()
    s = _slot(g, u, x)
    bad = dirs.copy()
    bad[s] = 3 if dirs[s] != 3 else 1
    _refused(g.row_ptr, g.col, bad, g.types)
    # the slot gone: an odd number of slots is refused on the host
    rp = g.row_ptr.copy()
    rp[u + 1:] -= 1
    _refused(rp, np.delete(g.col, s), np.delete(dirs, s), g.types, code=1)
    # moved to a node without the opposite: the number of slots stays even
    col = g.col.copy()
    b, e = int(rp[u]), int(g.row_ptr[u + 1])
    col[b:e] = np.sort(np.append(np.delete(col[b:e], s - b), 58))
    _refused(g.row_ptr, col, dirs, g.types)


@pytest.mark.parametrize("L", [1, 2, 16])
def test_class_runs(oracle_mod, L):
    rng = np.random.default_rng(L)
    n = 300
    rp, col = G.csr_from_edges(n, rng.integers(0, n, 2000), rng.integers(0, n, 2000))
    g = G.Graph(rp, col, rng.integers(0, L, n).astype(np.uint8), L, f"runs_L{L}")
    check(oracle_mod, g, G.orient(g, 0.2, L))
