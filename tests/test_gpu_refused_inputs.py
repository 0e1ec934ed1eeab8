"""Refused inputs of millions of slots: errors spread over the whole graph, so
that workgroups that start late find the status word already set by earlier
ones of their own kernel.  Every call returns its status and leaves its
outputs as they were."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N, REACH = 400_000, 5            # nodes, neighbours on each side: 4M slots


def _ring(n, reach=REACH):
    """Node u joined to u +- 1 .. reach (modulo n), rows sorted."""
    step = np.concatenate([np.arange(-reach, 0), np.arange(1, reach + 1)])
    col = np.sort((np.arange(n)[:, None] + step) % n, axis=1).astype(np.int32)
    rp = np.arange(n + 1, dtype=np.int64) * (2 * reach)
    return rp, col.reshape(-1), (np.arange(n) % 3).astype(np.uint8)


def _spoil(kind, n, reach=REACH):
    """The ring with every thousandth row spoiled, and the status it gets."""
    rp, col, types = _ring(n, reach)
    at = np.arange(500, n - 500, 1000)
    row = at * 2 * reach
    want = 2
    if kind == "unsorted":
        col[row], col[row + 1] = col[row + 1].copy(), col[row].copy()
    elif kind == "repeated":
        col[row + 1] = col[row]
    elif kind == "id":
        col[row + 2 * reach - 1] = n
    elif kind == "negative":
        col[row] = -1
    elif kind == "self_loop":
        col[row + reach] = at
    elif kind == "one_way":         # u -> u + reach + 1 instead of u + reach
        col[row + 2 * reach - 1] += 1
    elif kind == "offsets":
        rp[at + 1] = rp[at] - 1
    elif kind == "count":           # an entry below the diagonal taken above it
        col[row + reach - 1] = at + reach + 1
        for r in row:
            col[r:r + 2 * reach].sort()
    elif kind == "type":
        types[at] = 3
        want = 3
    return (rp, col, types), want


KINDS = ["unsorted", "repeated", "id", "negative", "self_loop", "one_way", "offsets", "count",
         "type"]


def _dev(arrays):
    import torch

    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def _code(call, *outs):
    """Status of the call; the outputs hold 77 before and, when it is refused,
    after."""
    import torch

    import paper_2010_14058_amd as P

    try:
        call()
    except P.TGError as e:
        torch.cuda.synchronize()
        assert all(bool((o == 77).all()) for o in outs)
        return e.code
    return 0


def _full(shape):
    import torch

    return torch.full(shape, 77, dtype=torch.int64, device="cuda")


@pytest.mark.parametrize("kind", KINDS)
def test_single_graph(kind):
    import paper_2010_14058_amd as P

    arrays, want = _spoil(kind, N)
    rp, col, types = _dev(arrays)
    print(f"[gpu] {kind}: n={N} nnz={col.numel()}", flush=True)
    glob, pa = _full((P.global_width(3),)), _full((P.pa_global_width(3),))
    assert _code(lambda: P.count_typed_graphlets(rp, col, types, 3, per_edge=False,
                                                 out_global=glob), glob) == want
    assert _code(lambda: P.count_position_aware(rp, col, types, 3, per_edge=False,
                                                out_global=pa), pa) == want


@pytest.mark.parametrize("kind", KINDS + ["direction", "no_direction"])
def test_directed(kind):
    import torch

    import paper_2010_14058_amd as P

    arrays, want = _spoil(kind, N)
    rp, col, types = _dev(arrays)
    dirs = torch.full((col.numel(),), 3, dtype=torch.uint8, device="cuda")
    if kind in ("direction", "no_direction"):
        dirs[::10_000] = 1 if kind == "direction" else 0
    print(f"[gpu] directed {kind}: n={N} nnz={col.numel()}", flush=True)
    assert _code(lambda: P.count_directed(rp, col, dirs, types, 3)) == want


def _batch_of_rings(kind, G, n, reach):
    """G rings of n nodes in one CSR, every fiftieth spoiled."""
    rp0, col0, types0 = _ring(n, reach)
    nnz = col0.size
    col = (np.tile(col0, (G, 1)) + (np.arange(G) * n)[:, None]).astype(np.int32)
    rp = np.concatenate([[0], (rp0[1:] + (np.arange(G) * nnz)[:, None]).reshape(-1)])
    types = np.tile(types0, G)
    bad = np.arange(7, G, 50)
    first = bad * n
    want = 2
    if kind == "unsorted":
        col[bad, 0], col[bad, 1] = col[bad, 1].copy(), col[bad, 0].copy()
    elif kind == "id":
        col[bad, -1] = G * n
    elif kind == "self_loop":
        col[bad, 0] = first
    elif kind == "one_way":         # an entry of the first node moved by one
        col[bad, reach] -= 1
    elif kind == "offsets":
        rp[first + 2] = rp[first + 1] - 1
    elif kind == "type":
        types[first] = 3
        want = 3
    elif kind == "cross":
        col[bad, 2 * reach - 1] = (first + n) % (G * n)
        want = 9
    node_ptr = np.arange(G + 1, dtype=np.int64) * n
    return (rp, col.reshape(-1), types), node_ptr, want


@pytest.mark.parametrize("rows", [False, True], ids=["small", "general"])
@pytest.mark.parametrize("kind", ["unsorted", "id", "self_loop", "one_way", "offsets", "type",
                                  "cross"])
def test_batch(kind, rows):
    import torch

    import paper_2010_14058_amd as P

    G, n, reach = 12_000, 24, 4
    arrays, node_ptr, want = _batch_of_rings(kind, G, n, reach)
    rp, col, types = _dev(arrays)
    plan = P.BatchPlan(rp, col, types, node_ptr, np.full(G, 3, np.int32))
    print(f"[gpu] batch {kind}: G={G} n={plan.n} nnz={plan.nnz} rows={rows}", flush=True)
    out, status = _full((int(plan.goff_host[-1]),)), _full((1,)).to(torch.int32)
    assert _code(lambda: P.count_batch(plan, per_edge=rows, out_globals=out), out) == want
    # without a host synchronisation: the status arrives on the device
    ws = P.Workspace("cuda")
    ws.get(P.batch_workspace_bytes(plan.n, plan.nnz, G, plan.L_max))
    out_rows = (torch.empty((plan.nnz // 2, P.row_width(3)), dtype=torch.int64, device="cuda")
                if rows else None)
    P.count_batch_async(plan, out, status, ws, torch.cuda.current_stream(), out_rows=out_rows)
    torch.cuda.synchronize()
    assert int(status.item()) == want
    assert bool((out == 77).all())


@pytest.mark.parametrize("rows", [False, True], ids=["small", "general"])
@pytest.mark.parametrize("G", [4, 4000])
def test_batch_error_order(G, rows):
    """An edge between two graphs is reported before a type out of range,
    whichever graph has which."""
    import paper_2010_14058_amd as P

    for typed in (0, 1, 2, G - 1):
        arrays, node_ptr, _ = _batch_of_rings("none", G, 24, 4)
        rp, col, types = arrays
        types[typed * 24 + 5] = 3
        col[1 * 24 * 8 + 7] = 2 * 24            # graph 1's first node joined to graph 2
        rp, col, types = _dev((rp, col, types))
        plan = P.BatchPlan(rp, col, types, node_ptr, np.full(G, 3, np.int32))
        print(f"[gpu] batch of {G}: a type in graph {typed}, an edge from 1 to 2", flush=True)
        assert _code(lambda: P.count_batch(plan, per_edge=rows)) == 9
