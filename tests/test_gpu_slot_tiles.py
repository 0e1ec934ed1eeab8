"""Flat walks of the adjacency (checks, edge ids, directed degrees) at sizes
where their tiles change: 256 slots up to 1,024 tiles of them, 512 and more
above, 2,048 at most.  Rings joined to their nearest nodes, so that every
edge's row follows from its length; one entry spoiled at the edge of a tile is
refused."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

REACH = 5


def _ring(n):
    step = np.concatenate([np.arange(-REACH, 0), np.arange(1, REACH + 1)])
    col = np.sort((np.arange(n)[:, None] + step) % n, axis=1).astype(np.int32)
    rp = np.arange(n + 1, dtype=np.int64) * (2 * REACH)
    return rp, col.reshape(-1), np.zeros(n, np.uint8)


def _general(rp, col, types):
    """Rows and global counts by the general kernels (graphs of few edges take
    them when a scheduling knob is off its default)."""
    import paper_2010_14058_amd as P

    old = P.set_tuning(clear_bytes=65)
    try:
        return P.count_typed_graphlets(rp, col, types, 1)
    finally:
        P.set_tuning(**old)


def _dev(arrays):
    import torch

    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def _length(n):
    """Circular distance of each canonical edge's ends."""
    rp, col, _ = _ring(n)
    src = np.repeat(np.arange(n), 2 * REACH)
    up = col > src
    d = (col - src)[up]
    return np.minimum(d, n - d)


@pytest.mark.parametrize("n", [26, 205, 26_214, 26_215, 52_500, 160_000])
def test_sizes(oracle_mod, n):
    import torch

    import paper_2010_14058_amd as P
    from tg_synth import graphs as G

    small = 24
    rp, col, types = _ring(small)
    want = oracle_mod.all_edge_rows(G.Graph(rp, col, types, 1, "ring"))
    by_len = {k: want[np.flatnonzero(_length(small) == k)[0]] for k in range(1, REACH + 1)}
    rp, col, types = _dev(_ring(n))
    print(f"[gpu] ring n={n} nnz={col.numel()}", flush=True)
    rows, _ = _general(rp, col, types)
    dirs = torch.full((col.numel(),), 3, dtype=torch.uint8, device="cuda")
    drows, _ = P.count_directed(rp, col, dirs, types, 1)
    torch.cuda.synchronize()
    rows, drows = rows.cpu().numpy(), drows.cpu().numpy()
    for k in range(1, REACH + 1):
        at = _length(n) == k
        np.testing.assert_array_equal(rows[at], np.broadcast_to(by_len[k].astype(np.int64),
                                                                rows[at].shape))
        # both directions everywhere: k's triangles and 2 * 10 - 2 - 2 T paths
        T = int(by_len[k][0])
        d = np.zeros(15, np.int64)
        d[8], d[9 + 2], d[12 + 2] = T, 2 * REACH - 1 - T, 2 * REACH - 1 - T
        np.testing.assert_array_equal(drows[at], np.broadcast_to(d, drows[at].shape))


@pytest.mark.parametrize("n,tile", [(205, 256), (26_214, 256), (52_500, 768), (160_000, 1792),
                                    (400_000, 2048)])
@pytest.mark.parametrize("kind", ["unsorted", "one_way"])
def test_refused_at_tile_edges(n, tile, kind):
    import torch

    import paper_2010_14058_amd as P

    def code(call):
        try:
            call()
        except P.TGError as e:
            return e.code
        return 0

    for t in (1, (n * 2 * REACH // tile) // 2):
        for slot in (t * tile - 1, t * tile):
            rp, col, types = _ring(n)
            u = slot // (2 * REACH)
            if kind == "unsorted":          # equal to its left neighbour in the row
                s = max(slot, u * 2 * REACH + 1)
                col[s] = col[s - 1]
            else:                           # the row's largest entry moved by one
                col[u * 2 * REACH + 2 * REACH - 1] += 1
            dirs = torch.full((col.size,), 3, dtype=torch.uint8, device="cuda")
            rp, col, types = _dev((rp, col, types))
            print(f"[gpu] {kind} at slot {slot} of {col.numel()}", flush=True)
            assert code(lambda: _general(rp, col, types)) == 2
            assert code(lambda: P.count_directed(rp, col, dirs, types, 1)) == 2
