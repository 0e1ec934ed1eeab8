"""Batches of small graphs counted graph by graph in LDS: global vectors
against the oracle at the edges of the size classes (64, 128, 256 and 512
nodes, where the bit rows and the sums change width), dense graphs (the
largest sums), few and many types, empty and edgeless graphs, and batches of
more graphs than the chip has workgroup slots."""

import numpy as np
import pytest

from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


def _batch(parts):
    offs = np.cumsum([0] + [p.n for p in parts]).astype(np.int64)
    rp = np.concatenate([np.zeros(1, np.int64)] + [
        p.row_ptr[1:] + b for p, b in zip(parts, np.cumsum([0] + [p.nnz for p in parts]))])
    col = np.concatenate([p.col + o for p, o in zip(parts, offs[:-1])] + [np.zeros(0, np.int32)])
    types = np.concatenate([p.types for p in parts])
    return rp, col.astype(np.int32), types, offs, np.array([p.L for p in parts], np.int32)


def _globals(parts):
    import torch

    import paper_2010_14058_amd as P

    rp, col, types, offs, L = _batch(parts)
    print(f"[gpu] batch of {len(parts)} graphs, n={offs[-1]} nnz={col.size}", flush=True)
    dev = torch.device("cuda:0")
    plan = P.BatchPlan(torch.from_numpy(rp).to(dev), torch.from_numpy(col).to(dev),
                       torch.from_numpy(types).to(dev), offs, L)
    glob, _ = P.count_batch(plan)
    torch.cuda.synchronize()
    return glob.cpu().numpy().view(np.uint64), plan.goff_host


def _check(oracle_mod, parts, which=None):
    got, off = _globals(parts)
    for g in range(len(parts)) if which is None else which:
        p = parts[g]
        want = (oracle_mod.global_counts(p, oracle_mod.all_edge_rows(p, threads=8)) if p.m
                else np.zeros(off[g + 1] - off[g], np.uint64))
        np.testing.assert_array_equal(got[off[g]:off[g + 1]], want, err_msg=f"graph {g}: {p.name}")


def _edgeless(n, L):
    return G.Graph(np.zeros(n + 1, np.int64), np.zeros(0, np.int32),
                   np.arange(n, dtype=np.uint8) % L, L, f"edgeless{n}")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512])
def test_class_edges(oracle_mod, n):
    parts = [G.random_small_graph(n, min(1.0, 8.0 / n), 5, 40 + n) if n > 2 else _edgeless(n, 2),
             _edgeless(0, 3), G.random_small_graph(9, 0.7, 3, n)]
    _check(oracle_mod, parts)


def test_dense_graphs(oracle_mod):
    # complete graphs of one type: the sums at their largest for the size
    parts = [G.random_small_graph(128, 1.1, 1, 1), G.random_small_graph(256, 1.1, 1, 2),
             G.random_small_graph(260, 1.1, 1, 3), G.random_small_graph(60, 0.9, 8, 4),
             G.random_small_graph(200, 0.4, 8, 5)]
    _check(oracle_mod, parts)


@pytest.mark.parametrize("L", [1, 4, 8, 10, 11, 16])
def test_types(oracle_mod, L):
    # 10 types and 512 nodes still fit a CU's LDS; 16 types with 300 nodes do
    # not and take the general path
    parts = [G.chung_lu_typed(300, 9.0, 2.2, 120.0, L, seed=L), G.random_small_graph(40, 0.3, L, 7),
             G.random_small_graph(100, 0.1, max(1, L - 1), 8)]
    _check(oracle_mod, parts)


def test_many_graphs(oracle_mod):
    b = G.batch_graphs(3000, seed=12)
    parts = [b.graph(g) for g in range(b.G)]
    _check(oracle_mod, parts, which=range(0, b.G, 37))


def test_refused_inputs():
    """What the general path refuses stays refused, and the outputs are left
    untouched."""
    import torch

    import paper_2010_14058_amd as P

    good = _batch([G.random_small_graph(20, 0.4, 3, 1), G.random_small_graph(30, 0.3, 3, 2)])
    dev = torch.device("cuda:0")

    def status(rp=None, col=None, types=None):
        a = [x if y is None else y for x, y in zip(good, (rp, col, types, None, None))]
        plan = P.BatchPlan(*(torch.from_numpy(np.ascontiguousarray(x)).to(dev) for x in a[:3]),
                           a[3], a[4])
        out = torch.full((int(plan.goff_host[-1]),), 77, dtype=torch.int64, device=dev)
        try:
            P.count_batch(plan, out_globals=out)
        except P.TGError as e:
            assert bool((out == 77).all())
            return e.code
        return 0

    rp, col, types = good[:3]
    assert status() == 0
    for bad, want in ((-1, 2), (50, 2), (25, 9)):      # id below 0, above n, in another graph
        c = col.copy()
        c[0] = bad
        assert status(col=c) == want
    u = int(np.flatnonzero(np.diff(rp) >= 2)[0])
    c = col.copy()
    c[rp[u]:rp[u] + 2] = c[rp[u]:rp[u] + 2][::-1]      # unsorted row
    assert status(col=c) == 2
    c = col.copy()
    c[rp[u] + 1] = c[rp[u]]                            # a neighbour twice
    assert status(col=c) == 2
    t = types.copy()
    t[-1] = 3
    assert status(types=t) == 3
    # 0-1 present one way only: move node 0's first neighbour to another id
    row = set(col[rp[0]:rp[1]].tolist())
    first = int(col[0])
    other = next(x for x in range(1, 20) if x not in row and x < col[1] and x != first)
    c = col.copy()
    c[0] = other
    assert status(col=c) == 2
    r = rp.copy()
    r[3], r[4] = r[4], r[3]                            # decreasing row offsets
    assert r[3] == r[4] or status(rp=r) == 2
