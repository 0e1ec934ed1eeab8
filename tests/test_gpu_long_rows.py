"""The passes flat over the adjacency and the long rows taken by workgroups:
rows of the long-row degree (1023 to 1025), a row over many tiles of slots, and
tiles that span more rows than are staged in LDS (mostly isolated nodes), for
undirected and directed counts, against the oracle."""

import numpy as np
import pytest

from gpu_util import run_gpu
from test_gpu_directed import check as check_directed
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


def _graph(n, hubs, extra, L, seed, lo=0):
    """hubs: degree of node q for q = 0, 1, ...; extra random pairs above lo."""
    rng = np.random.default_rng(seed)
    u = [np.full(d, q) for q, d in enumerate(hubs)]
    v = [rng.choice(np.arange(len(hubs), n), d, replace=False) for d in hubs]
    u.append(rng.integers(lo, n, extra))
    v.append(rng.integers(lo, n, extra))
    rp, col = G.csr_from_edges(n, np.concatenate(u), np.concatenate(v))
    return G.Graph(rp, col, rng.integers(0, L, n).astype(np.uint8), L, f"rows_n{n}_L{L}")


def _check(oracle_mod, g):
    rows, glob = run_gpu(g)
    want = oracle_mod.all_edge_rows(g, threads=8)
    np.testing.assert_array_equal(rows, want)
    np.testing.assert_array_equal(glob, oracle_mod.global_counts(g, want))


@pytest.mark.parametrize("L", [1, 5, 16])
def test_long_row_degrees(oracle_mod, L):
    g = _graph(9000, [1022, 1023, 1024, 1025, 5000], 6000, L, 3, lo=2000)
    assert g.n > 8192
    _check(oracle_mod, g)


def test_sparse_tiles(oracle_mod):
    # 40,000 nodes, 4,000 edges: a tile of 2,048 slots covers thousands of rows
    g = _graph(40_000, [], 4000, 3, 4)
    _check(oracle_mod, g)
    check_directed(oracle_mod, g, G.orient(g, 0.3, 5))


def test_directed_hub(oracle_mod):
    g = _graph(6000, [5000, 1024], 3000, 4, 6, lo=2)
    check_directed(oracle_mod, g, G.orient(g, 0.2, 7))


def test_unsorted_across_tiles():
    """A row over several tiles with one pair out of order, at a tile's edge."""
    import torch

    import paper_2010_14058_amd as P

    g = _graph(6000, [5000], 12_000, 2, 8, lo=1)
    dev = torch.device("cuda:0")
    rp, ty = torch.from_numpy(g.row_ptr).to(dev), torch.from_numpy(g.types).to(dev)
    old = P.set_tuning(clear_bytes=65)      # the general pipeline for this small graph
    try:
        for at in (1, 2047, 2048, 4096, 4999):
            col = g.col.copy()
            col[at - 1], col[at] = col[at], col[at - 1]
            with pytest.raises(P.TGError) as e:
                P.count_typed_graphlets(rp, torch.from_numpy(col).to(dev), ty, 2)
            assert e.value.code == 2
    finally:
        P.set_tuning(**old)
