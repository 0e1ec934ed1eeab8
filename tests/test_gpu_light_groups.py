"""Light 4-cycle groups at the bounds of their tables: groups of 127 to 129 and
511 to 513 wedges (in few items, and in more than 64 items), the same group
sizes with the light bucket lowered to and around the small table's bound."""

import numpy as np
import pytest

from gpu_util import run_gpu
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


def _bipartite(sizes, L, seed):
    """For each (a, b): a centres joined to a top node and to b targets each,
    targets drawn from a pool; every piece is its own component."""
    rng = np.random.default_rng(seed)
    u, v, n = [], [], 0
    for a, b in sizes:
        top, centres = n, n + 1 + np.arange(a)
        pool = n + 1 + a + np.arange(b + 3)
        n = int(pool[-1]) + 1
        # leaves raise the top node's degree above every centre's
        leaves = n + np.arange(b + 40)
        n = int(leaves[-1]) + 1
        u += [np.full(a, top), np.full(leaves.size, top)]
        v += [centres, leaves]
        for c in centres:
            u.append(np.full(b, c))
            v.append(rng.choice(pool, b, replace=False))
    rp, col = G.csr_from_edges(n, np.concatenate(u), np.concatenate(v))
    return G.Graph(rp, col, rng.integers(0, L, n).astype(np.uint8), L, f"groups_L{L}")


SIZES = [(1, 127), (2, 64), (3, 43), (127, 1), (128, 1), (129, 1), (64, 2), (65, 2), (8, 16),
         (7, 73), (8, 64), (9, 57), (511, 1), (512, 1), (171, 3), (73, 7)]


@pytest.mark.parametrize("L", [1, 4, 16])
@pytest.mark.parametrize("light", [512, 129, 128, 127, 1])
def test_group_sizes(oracle_mod, L, light):
    import paper_2010_14058_amd as P

    g = _bipartite(SIZES, L, 5)
    old = P.set_tuning(light_wedges=light, clear_bytes=65)
    try:
        rows, glob = run_gpu(g)
    finally:
        P.set_tuning(**old)
    want = oracle_mod.all_edge_rows(g, threads=8)
    np.testing.assert_array_equal(rows, want)
    np.testing.assert_array_equal(glob, oracle_mod.global_counts(g, want))
