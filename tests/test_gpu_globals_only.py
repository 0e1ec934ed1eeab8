"""Global counts without the per-edge table (sums of not necessarily induced
copies) against those that come with it, and against the oracle: power laws
with hub cores and super-hubs, a tripartite graph, dense graphs (many cliques
among hubs and among low nodes), 1 to 8 types (and 9, which keep the per-edge
pipeline), every 4-cycle path (light, task and blocked groups)."""

import numpy as np
import pytest

from gpu_util import run_gpu
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


def _check(g, oracle_mod=None, **knobs):
    import paper_2010_14058_amd as P

    old = P.set_tuning(**dict(dict(clear_bytes=65), **knobs))
    try:
        _, full = run_gpu(g)
        _, only = run_gpu(g, per_edge=False)
    finally:
        P.set_tuning(**old)
    np.testing.assert_array_equal(only, full)
    if oracle_mod is not None:
        want = oracle_mod.global_counts(g, oracle_mod.all_edge_rows(g, threads=8))
        np.testing.assert_array_equal(only, want)


@pytest.mark.parametrize("L", [1, 2, 3, 5, 6, 7, 8, 9])
def test_types(oracle_mod, L):
    _check(G.chung_lu_typed(4000, 12.0, 2.1, 900.0, L, seed=L, name=f"cl4k_L{L}"), oracle_mod)


@pytest.mark.parametrize("knobs", [dict(), dict(sh_deg=32), dict(sh_max=0),
                                   dict(light_wedges=1), dict(blk_wedges=1, light_wedges=1),
                                   dict(blk_wedges=1, blk_task=1024), dict(task_wedges=64),
                                   dict(light_wedges=64)],
                         ids=["default", "superhubs", "no_superhubs", "no_light", "all_blocked",
                              "small_tasks", "split_tasks", "small_light"])
def test_paths(knobs):
    _check(G.chung_lu_typed(20000, 16.0, 2.1, 3000.0, 5, type_probs=G.zipf_probs(5, 1.2),
                            homophily=0.6, seed=5, name="cl_20k"), **knobs)


def test_hub_core_overflow():
    # more nodes of degree 32 than the hub core takes: cliques of low nodes, of
    # low nodes with hubs, and of more hubs than are tested pair by pair
    _check(G.chung_lu_typed(14000, 60.0, 2.3, 4000.0, 4, seed=9, name="cl_dense"))


@pytest.mark.parametrize("n,p", [(60, 1.1), (150, 0.5), (400, 0.3), (31, 1.1)])
def test_dense(oracle_mod, n, p):
    # every node in the hub core, or none (degree below 32)
    _check(G.random_small_graph(n, p, 4, n), oracle_mod)


def test_tripartite_and_sparse():
    _check(G.config_graph(3, scale=0.02))
    _check(G.er_graph(12000, 3.0, 3, seed=2))


def test_degree_above_16_bits():
    rng = np.random.default_rng(4)
    n = 70_002
    u = np.concatenate([np.zeros(70_000, np.int64), rng.integers(1, n, 90_000)])
    v = np.concatenate([np.arange(1, 70_001), rng.integers(1, n, 90_000)])
    rp, col = G.csr_from_edges(n, u, v)
    _check(G.Graph(rp, col, rng.integers(0, 3, n).astype(np.uint8), 3, "hub70k"))
