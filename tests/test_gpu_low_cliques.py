"""4-cliques below the hub core without per-edge rows: complete graphs whose
edges have up to 64, 65, 256 and 257 members (the edges of the lists in LDS)
beside 8,192 nodes of higher degree, against the sums of the per-edge rows."""

import numpy as np
import pytest

from gpu_util import run_gpu
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [4, 66, 67, 258, 259])
@pytest.mark.parametrize("L", [1, 3])
def test_members(q, L):
    hubs, reach = 8192, 140
    u = np.repeat(np.arange(hubs), reach)
    v = (u + np.tile(np.arange(1, reach + 1), hubs)) % hubs
    a, b = np.triu_indices(q, 1)
    # a few edges from the complete graph to the hubs: members of both kinds
    x = np.arange(0, q, 3)
    rp, col = G.csr_from_edges(hubs + q, np.concatenate([u, hubs + a, hubs + x]),
                               np.concatenate([v, hubs + b, np.zeros_like(x)]))
    types = np.random.default_rng(q).integers(0, L, hubs + q).astype(np.uint8)
    g = G.Graph(rp, col, types, L, f"K{q}_beside_hubs_L{L}")
    rows, glob = run_gpu(g)
    _, glob2 = run_gpu(g, per_edge=False)
    np.testing.assert_array_equal(glob2, glob)
    # every edge's cliques, six edges each
    assert int(rows[:, -(L * (L + 1) // 2):].sum()) == 6 * int(glob[-len(_k4(L)):].sum())


def _k4(L):
    import math

    return range(math.comb(L + 3, 4))
