"""Edges by their triangles (none, up to 16, more) and smaller degree (up to
256, more): graphs with edges on both sides of each bound, with and without
hub-core and super-hub endpoints, against the oracle."""

import numpy as np
import pytest

from gpu_util import run_gpu
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


def _graph(n, u, v, L, seed, name):
    rp, col = G.csr_from_edges(n, np.concatenate(u), np.concatenate(v))
    types = np.random.default_rng(seed).integers(0, L, n).astype(np.uint8)
    return G.Graph(rp, col, types, L, name)


def _check(oracle_mod, g, knobs):
    import paper_2010_14058_amd as P

    old = P.set_tuning(**knobs)
    try:
        rows, glob = run_gpu(g)
    finally:
        P.set_tuning(**old)
    want = oracle_mod.all_edge_rows(g, threads=8)
    np.testing.assert_array_equal(rows, want)
    np.testing.assert_array_equal(glob, oracle_mod.global_counts(g, want))


# a knob off its default keeps small graphs on the general pipeline; the
# second set makes every node of degree 32 or more a super-hub
KNOBS = [dict(clear_bytes=65), dict(sh_deg=32)]


@pytest.mark.parametrize("knobs", KNOBS, ids=["hub_core", "superhubs"])
@pytest.mark.parametrize("L", [1, 3, 5, 8, 9, 16])
def test_triangle_bounds(oracle_mod, L, knobs):
    # books: an edge with exactly t pages is in t triangles (15, 16, 17 and
    # others); every second page joined to the next, so some pages are in
    # cliques with the spine
    u, v, n = [], [], 0
    for t in (0, 1, 2, 7, 8, 9, 15, 16, 17, 40):
        a, b, pages = n, n + 1, np.arange(n + 2, n + 2 + t)
        u += [np.array([a]), np.full(t, a), np.full(t, b), pages[:-1:2] if t > 1 else pages[:0]]
        v += [np.array([b]), pages, pages, pages[1::2] if t > 1 else pages[:0]]
        n += 2 + t
    rng = np.random.default_rng(L)
    u.append(rng.integers(0, n, 200))
    v.append(rng.integers(0, n, 200))
    _check(oracle_mod, _graph(n, u, v, L, 5, f"books_L{L}"), knobs)


@pytest.mark.parametrize("knobs", KNOBS, ids=["hub_core", "superhubs"])
@pytest.mark.parametrize("deg", [255, 256, 257])
def test_degree_bound(oracle_mod, deg, knobs):
    # two joined nodes of the given degree with five common neighbours
    common = np.arange(2, 7)
    own = deg - 1 - common.size
    la = np.arange(7, 7 + own)
    lb = la + own
    n = int(lb[-1]) + 1
    u = [np.array([0]), np.zeros(5, np.int64), np.ones(5, np.int64), np.zeros(own, np.int64),
         np.ones(own, np.int64), common[:-1]]
    v = [np.array([1]), common, common, la, lb, common[1:]]
    rng = np.random.default_rng(deg)
    u.append(rng.integers(7, n, 300))
    v.append(rng.integers(7, n, 300))
    _check(oracle_mod, _graph(n, u, v, 4, 6, f"pair_{deg}"), knobs)


@pytest.mark.parametrize("m", [1, 7, 8, 9, 1023, 1024, 1025])
def test_list_ends(oracle_mod, m):
    # few edges of every class: m edges of a dense or sparse random graph
    n = max(3, int(1.6 * np.sqrt(m)) + 2)
    rng = np.random.default_rng(m)
    iu, ju = np.triu_indices(n, 1)
    pick = rng.choice(iu.size, size=min(m, iu.size), replace=False)
    _check(oracle_mod, _graph(n, [iu[pick]], [ju[pick]], 3, 7, f"m{m}"), KNOBS[0])
