"""Global sums of single graphs whose histogram exceeds LDS (ten types and
more): in copies in the 4-cycle maps' space, few of them or none where the maps
are small.  Rows and global counts against the oracle, by the general kernels
(a scheduling knob off its default)."""

import numpy as np
import pytest

from gpu_util import run_gpu
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [2048, 9, 1], ids=["16_copies", "few", "none"])
@pytest.mark.parametrize("L", [9, 10, 16])
def test_copies(oracle_mod, L, slots):
    import paper_2010_14058_amd as P

    # nine maps of n * L / 2 words hold eight copies (L = 10) or two (16), one
    # map none
    n = {9: 900, 10: 900, 16: 1200}[L]
    g = G.chung_lu_typed(n, 10.0, 2.1, 150.0, L, seed=L, name=f"cl_L{L}")
    old = P.set_tuning(clear_bytes=65, cycle_slots=slots)
    try:
        rows, glob = run_gpu(g)
        _, glob2 = run_gpu(g, per_edge=False)
    finally:
        P.set_tuning(**old)
    want = oracle_mod.all_edge_rows(g, threads=8)
    np.testing.assert_array_equal(rows, want)
    np.testing.assert_array_equal(glob, oracle_mod.global_counts(g, want))
    np.testing.assert_array_equal(glob2, glob)
