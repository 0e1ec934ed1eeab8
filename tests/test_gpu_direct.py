"""Single graphs counted edge by edge from their own neighbourhoods, against
the oracle at the edges of that path's range (largest degree, node count, walk
length, types, alignment of the types) and against the general pipeline, which
a scheduling knob off its default selects."""

import numpy as np
import pytest

from gpu_util import run_gpu
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


def _general(g, **kw):
    import paper_2010_14058_amd as P

    old = P.set_tuning(clear_bytes=65)
    try:
        return run_gpu(g, **kw)
    finally:
        P.set_tuning(**old)


def _took_direct():
    import paper_2010_14058_amd as P

    return sum(P.last_stats().values()) == 0


def _star(leaves, n, L, extra=40, seed=3):
    rng = np.random.default_rng(seed)
    u = np.concatenate([np.zeros(leaves, np.int64), rng.integers(1, n, extra)])
    v = np.concatenate([np.arange(1, leaves + 1), rng.integers(1, n, extra)])
    rp, col = G.csr_from_edges(n, u, v)
    return G.Graph(rp, col, rng.integers(0, L, n).astype(np.uint8), L, f"star{leaves}")


def _check(oracle_mod, g):
    rows, glob = run_gpu(g)
    took = _took_direct()
    want = oracle_mod.all_edge_rows(g, threads=8)
    np.testing.assert_array_equal(rows, want)
    np.testing.assert_array_equal(glob, oracle_mod.global_counts(g, want))
    _, only = run_gpu(g, per_edge=False)
    np.testing.assert_array_equal(only, glob)
    grows, gglob = _general(g)
    assert not _took_direct()
    np.testing.assert_array_equal(grows, rows)
    np.testing.assert_array_equal(gglob, glob)
    return took


@pytest.mark.parametrize("L", [1, 5, 10, 16])
def test_types(oracle_mod, L):
    # ten types are the last whose global sums fit the workgroup's LDS share
    assert _check(oracle_mod, G.chung_lu_typed(400, 9.0, 2.2, 90.0, L, seed=L))


@pytest.mark.parametrize("leaves,direct", [(511, True), (512, True), (513, False)])
def test_largest_degree(oracle_mod, leaves, direct):
    assert _check(oracle_mod, _star(leaves, 700, 3)) == direct


@pytest.mark.parametrize("n,direct", [(8191, True), (8192, True), (8193, False)])
def test_most_nodes(oracle_mod, n, direct):
    assert _check(oracle_mod, _star(30, n, 4, extra=3000)) == direct


def test_dense_and_long_walk(oracle_mod):
    assert _check(oracle_mod, G.random_small_graph(65, 1.1, 4, 1))       # complete: every pair near
    # 2^27 steps and more are left to the general pipeline
    assert not _check(oracle_mod, G.random_small_graph(200, 0.9, 2, 2))


def test_unaligned_types():
    import torch

    import paper_2010_14058_amd as P

    g = G.chung_lu_typed(301, 8.0, 2.2, 60.0, 3, seed=4)
    want, wg = run_gpu(g)
    dev = torch.device("cuda:0")
    rp, col = torch.from_numpy(g.row_ptr).to(dev), torch.from_numpy(g.col).to(dev)
    for shift in (1, 2, 3):
        buf = torch.zeros(g.n + 4, dtype=torch.uint8, device=dev)
        ty = buf[shift:shift + g.n]
        ty.copy_(torch.from_numpy(g.types))
        rows, glob = P.count_typed_graphlets(rp, col, ty, 3)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(rows.cpu().numpy().view(np.uint64), want)
        np.testing.assert_array_equal(glob.cpu().numpy().view(np.uint64), wg)


def test_refused_leaves_outputs():
    """An input error is found before any output is written."""
    import torch

    import paper_2010_14058_amd as P

    g = G.random_small_graph(30, 0.3, 2, 5)
    dev = torch.device("cuda:0")
    rows = torch.full((g.m, P.row_width(2)), 77, dtype=torch.int64, device=dev)
    glob = torch.full((P.global_width(2),), 77, dtype=torch.int64, device=dev)
    u = int(np.flatnonzero(np.diff(g.row_ptr) >= 2)[0])
    row = set(g.col[g.row_ptr[u]:g.row_ptr[u + 1]].tolist()) | {u}
    col = g.col.copy()
    last = int(g.row_ptr[u + 1]) - 1
    col[last] = next(x for x in range(29, -1, -1) if x not in row)   # its mirror is missing
    col[int(g.row_ptr[u]):last + 1].sort()
    types = g.types.copy()
    types[7] = 2
    for c, t, want in ((col, g.types, 2), (g.col, types, 3)):
        with pytest.raises(P.TGError) as e:
            P.count_typed_graphlets(torch.from_numpy(g.row_ptr).to(dev),
                                    torch.from_numpy(c).to(dev), torch.from_numpy(t).to(dev), 2,
                                    out_rows=rows, out_global=glob)
        assert e.value.code == want
        assert bool((rows == 77).all()) and bool((glob == 77).all())
