"""Components at the edges of the row partials (32 rows up to 8,192 of them,
64 above) with rows at and past the nonzeros of one item (128, 129, 641):
eigenpairs of the edge-weighted graph against scipy.  The solver stops at
||M x - theta x|| <= 1e-12 with M = I - L / 2, so ||L x - lambda x|| is at most
2e-12 plus the rounding of the host's products: 1e-11."""

import numpy as np
import pytest

from gpu_util import device
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [96, 97, 2048, 8192, 8193])
def test_partials(n):
    import scipy.sparse as sp
    import scipy.sparse.linalg as sla
    import torch

    import paper_2010_14058_amd as P

    rng = np.random.default_rng(n)
    k, per = 4, n // 4
    # four blocks of about 12 neighbours a node, a few edges between them
    u = rng.integers(0, n, 6 * n)
    v = np.minimum((u // per) * per + rng.integers(0, per, 6 * n), n - 1)
    x = rng.integers(0, n, (2, n // 8))
    us, vs = [u, np.arange(n), x[0]], [v, (np.arange(n) + 1) % n, x[1]]
    for q, d in enumerate((118, 119, 631)):
        if 2 * d < per:
            us.append(np.full(d, q * per))
            vs.append(q * per + rng.choice(np.arange(1, per), d, replace=False))
    rp, col = G.csr_from_edges(n, np.concatenate(us), np.concatenate(vs))
    m = col.shape[0] // 2
    print(f"[gpu] embedding n={n} m={m} max degree {np.diff(rp).max()}", flush=True)
    U, ev, comp, _ = P.graphlet_embedding(
        torch.from_numpy(rp).to(device()), torch.from_numpy(col).to(device()),
        torch.ones(m, dtype=torch.int64, device=device()), k, raw=True, tol=1e-12)
    torch.cuda.synchronize()
    U, ev, comp = U.cpu().numpy(), ev.cpu().numpy(), comp.cpu().numpy()
    assert not comp.any()               # one component, named by node 0
    A = sp.csr_matrix((np.ones(2 * m), col, rp), shape=(n, n))
    s = sp.diags(1.0 / np.sqrt(np.diff(rp)))
    S = s @ A @ s
    lam = ev[0]
    want = np.sort(1.0 - sla.eigsh(S, k=k, which="LA", tol=1e-13, return_eigenvectors=False))
    np.testing.assert_allclose(lam, want, rtol=0, atol=1e-9)
    np.testing.assert_allclose(U.T @ U, np.eye(k), rtol=0, atol=1e-10)
    assert np.linalg.norm(U - S @ U - U * lam, axis=0).max() <= 1e-11


@pytest.mark.parametrize("deg", [127, 128, 129, 256, 257])
def test_long_rows(deg):
    """A star: L has eigenvalues 0, 1 (deg - 1 times) and 2; the hub's row is
    one item or several."""
    import torch

    import paper_2010_14058_amd as P

    n = deg + 1
    rp, col = G.csr_from_edges(n, np.zeros(deg, dtype=np.int64), np.arange(1, n))
    U, ev, comp, _ = P.graphlet_embedding(
        torch.from_numpy(rp).to(device()), torch.from_numpy(col).to(device()),
        torch.ones(deg, dtype=torch.int64, device=device()), 1, raw=True, tol=1e-12)
    torch.cuda.synchronize()
    # the first eigenvector: the square roots of the degrees
    want = np.sqrt(np.diff(rp) / (2.0 * deg))
    got = U.cpu().numpy()[:, 0]
    np.testing.assert_allclose(ev.cpu().numpy()[0, 0], 0.0, atol=1e-12)
    np.testing.assert_allclose(got * np.sign(got[0]), want, rtol=0, atol=1e-10)
