"""Edges whose shorter row is at the bound above which a whole wave walks it
(128, 129) or well past it, next to short ones in the same wave, for both
unrolled numbers of types, against the oracle."""

import numpy as np
import pytest

from gpu_util import run_gpu
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("knobs", [dict(clear_bytes=65), dict(sh_deg=64)],
                         ids=["hub_core", "superhubs"])
@pytest.mark.parametrize("L", [1, 8, 9, 16])
def test_wave_rows(oracle_mod, L, knobs):
    import paper_2010_14058_amd as P

    # a clique on k nodes (degree k - 1), every second one with a leaf more,
    # and a random part below the bound
    k, extra, big = 129, 900, 200
    iu, iv = np.triu_indices(k, 1)
    leaves = np.arange(0, k, 2)
    rng = np.random.default_rng(L)
    ru, rv = rng.integers(400, 700, extra), rng.integers(400, 700, extra)
    n = 1000
    u = np.concatenate([iu, leaves, ru, np.full(big, 399), np.full(big, 398)])
    v = np.concatenate([iv, 200 + leaves, rv, 700 + np.arange(big), 700 + np.arange(big)])
    u, v = np.append(u, 398), np.append(v, 399)      # two rows of 201, 200 triangles
    rp, col = G.csr_from_edges(n, u, v)
    g = G.Graph(rp, col, rng.integers(0, L, n).astype(np.uint8), L, f"wave_rows_L{L}")
    deg = np.diff(rp)
    assert {128, 129, 201} <= set(deg.tolist())
    old = P.set_tuning(**knobs)
    try:
        rows, glob = run_gpu(g)
    finally:
        P.set_tuning(**old)
    want = oracle_mod.all_edge_rows(g, threads=8)
    np.testing.assert_array_equal(rows, want)
    np.testing.assert_array_equal(glob, oracle_mod.global_counts(g, want))
