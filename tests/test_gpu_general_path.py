"""The general kernels on graphs so small that other paths take them by
default: a scheduling knob off its default (single graphs), or per-edge rows or
a graph of more than 512 nodes (batches)."""

import numpy as np
import pytest

from gpu_util import run_gpu, to_device
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


@pytest.fixture
def general():
    import paper_2010_14058_amd as P

    old = P.set_tuning(clear_bytes=65)
    yield P
    P.set_tuning(**old)


# (row offsets, neighbours, types), status; the first is the path 0-1-2-3
PATH = ([0, 1, 3, 5, 6], [1, 0, 2, 1, 3, 2], [0, 1, 0, 1])
REFUSED = {
    "type": (PATH[0], PATH[1], [0, 1, 2, 1], 3),
    "self_loop": (PATH[0], [1, 1, 2, 1, 3, 2], PATH[2], 2),
    "unsorted": (PATH[0], [1, 2, 0, 1, 3, 2], PATH[2], 2),
    "repeated": (PATH[0], [1, 0, 0, 1, 3, 2], PATH[2], 2),
    "id": (PATH[0], [1, 0, 2, 1, 9, 2], PATH[2], 2),
    "negative": (PATH[0], [1, -1, 2, 1, 3, 2], PATH[2], 2),
    "offsets_fall": ([0, 1, 5, 3, 6], PATH[1], PATH[2], 2),
    "offsets_start": ([1, 1, 3, 5, 6], PATH[1], PATH[2], 2),
    "offsets_end": ([0, 1, 3, 5, 5], PATH[1], PATH[2], 2),
    "offsets_past": ([0, 1, 3, 9, 6], PATH[1], PATH[2], 2),
    "edge_count": ([0, 1, 2, 3, 4], [1, 2, 3, 2], PATH[2], 2),
    "one_way": ([0, 1, 1, 1, 2], [1, 2], PATH[2], 2),
    "type_and_loop": (PATH[0], [1, 1, 2, 1, 3, 2], [0, 1, 2, 1], 3),
}


def _arrays(rp, col, types):
    return (np.array(rp, np.int64), np.array(col, np.int32), np.array(types, np.uint8))


def _refused(P, call, *outs):
    with pytest.raises(P.TGError) as e:
        call()
    assert all(bool((o == 77).all()) for o in outs)
    return e.value.code


@pytest.mark.parametrize("case", list(REFUSED))
def test_refused(general, case):
    import torch

    P = general
    rp, col, types, want = REFUSED[case]
    a = to_device(G.Graph(*_arrays(rp, col, types), 2, case))
    glob = torch.full((P.global_width(2),), 77, dtype=torch.int64, device="cuda")
    rows = torch.full((len(col) // 2, P.row_width(2)), 77, dtype=torch.int64, device="cuda")
    assert _refused(P, lambda: P.count_typed_graphlets(*a, 2, out_rows=rows, out_global=glob),
                    rows, glob) == want
    assert _refused(P, lambda: P.count_typed_graphlets(*a, 2, per_edge=False, out_global=glob),
                    glob) == want
    glob = torch.full((P.pa_global_width(2),), 77, dtype=torch.int64, device="cuda")
    assert _refused(P, lambda: P.count_position_aware(*a, 2, out_global=glob), glob) == want


@pytest.mark.parametrize("rows", [True, False], ids=["rows", "wide"])
@pytest.mark.parametrize("case", list(REFUSED) + ["cross"])
def test_refused_batch(case, rows):
    """The malformed graph second in a batch; without rows beside a graph of 513
    nodes."""
    import torch

    import paper_2010_14058_amd as P

    first = G.random_small_graph(513 if not rows else 30, 0.02 if not rows else 0.2, 2, 5)
    if case == "cross":
        rp, col, types, want = *PATH, 9
        col = [1, 0, 2, 1, 3, 2]
    else:
        rp, col, types, want = REFUSED[case]
    rp, col, types = _arrays(rp, col, types)
    inside = (col >= 0) & (col < 4)
    col = np.where(inside, col + first.n, np.where(col < 0, -1, first.n + 99)).astype(np.int32)
    if case == "cross":
        col[0] = 3                   # the path's first node joined to the first graph
    n = first.n + 4
    rp = np.concatenate([first.row_ptr[:-1], rp + first.nnz])
    if case == "offsets_start":
        rp[0] = 1
    arrays = (rp, np.concatenate([first.col, col]), np.concatenate([first.types, types]))
    a = to_device(G.Graph(*arrays, 2, case))
    plan = P.BatchPlan(*a, np.array([0, first.n, n]), np.array([2, 2], np.int32))
    out = torch.full((int(plan.goff_host[-1]),), 77, dtype=torch.int64, device="cuda")
    assert _refused(P, lambda: P.count_batch(plan, per_edge=rows, out_globals=out), out) == want


@pytest.mark.parametrize("knobs", [dict(light_wedges=1, edge_deg=1),
                                   dict(light_wedges=64, edge_deg=16),
                                   dict(light_wedges=512, edge_deg=1024)],
                         ids=["all_heavy", "small_buckets", "largest_buckets"])
def test_degree_buckets(oracle_mod, general, knobs):
    """The degree buckets of 4-cycle groups and edges, in the kernels that have
    them: a single graph, and a batch with its rows."""
    P = general
    old = P.set_tuning(**knobs)
    try:
        g = G.chung_lu_typed(4000, 10.0, 2.1, 600.0, 4, seed=21, name="cl_4k_buckets")
        rows, glob = run_gpu(g)
        st = P.last_stats()
        want = oracle_mod.all_edge_rows(g, threads=8)
        np.testing.assert_array_equal(rows, want)
        np.testing.assert_array_equal(glob, oracle_mod.global_counts(g, want))
        d, uv = g.degrees(), g.edges()
        assert st["wedges_pass_a"] > 0 and st["light_groups"] > 0
        assert st["heavy_edges"] == int(np.sum(np.minimum(d[uv[:, 0]], d[uv[:, 1]]) >
                                               knobs["edge_deg"]))
        b = G.batch_graphs(60, seed=4)
        u = b.union
        plan = P.BatchPlan(*to_device(u), b.node_ptr, b.L)
        glob, rows = P.count_batch(plan, per_edge=True)
        glob = glob.cpu().numpy().view(np.uint64)
        st = P.last_stats()
        d, uv = u.degrees(), u.edges()
        assert st["wedges_pass_a"] > 0
        assert st["heavy_edges"] == int(np.sum(np.minimum(d[uv[:, 0]], d[uv[:, 1]]) >
                                               knobs["edge_deg"]))
        for q in range(b.G):
            gg = b.graph(q)
            want = oracle_mod.global_counts(gg, oracle_mod.all_edge_rows(gg))
            np.testing.assert_array_equal(glob[plan.goff_host[q]:plan.goff_host[q + 1]], want)
    finally:
        P.set_tuning(**old)
