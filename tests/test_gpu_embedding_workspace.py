"""Components of many long rows within the workspace that is asked for: all
rows longer than one item (128 nonzeros), so that items of 256 (200 nodes:
rows of 199) or 512 (300 and 600 nodes) are taken; nothing past the workspace
is written."""

import numpy as np
import pytest

from gpu_util import device
from tg_synth import graphs as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [200, 300, 600])
def test_dense_component(n):
    import torch

    import paper_2010_14058_amd as P

    dim, guard = 8, 1 << 16
    u, v = np.triu_indices(n, 1)
    rp, col = G.csr_from_edges(n, u, v)
    rng = np.random.default_rng(n)
    # ten groups of strong edges: the wanted eigenvalues lie apart from the rest
    w = rng.integers(1, 10, u.size) + np.where(u % 10 == v % 10, 5000, 0)
    print(f"[gpu] embedding of a complete graph, n={n}", flush=True)
    need = P._lib.load().tg_embedding_workspace_bytes(n, col.size, dim)
    ws = P.Workspace(device())
    ws.get(need + guard)
    ws.buf[need:] = 0xA5

    class Exact:
        def get(self, nbytes):
            assert nbytes == need
            return ws.buf[:need]

    _, ev, comp, _ = P.graphlet_embedding(
        torch.from_numpy(rp).to(device()), torch.from_numpy(col).to(device()),
        torch.from_numpy(w.astype(np.int64)).to(device()), dim, workspace=Exact())
    torch.cuda.synchronize()
    assert bool((ws.buf[need:] == 0xA5).all())
    assert not comp.cpu().numpy().any()
    W = np.zeros((n, n))
    W[u, v] = W[v, u] = w
    d = 1.0 / np.sqrt(W.sum(1))
    want = np.linalg.eigvalsh(np.eye(n) - d[:, None] * W * d[None, :])[:dim]
    # the solver stops at a residual of 1e-10 of (S + I) / 2: eigenvalues
    # within 2e-10, and the host's rounding
    np.testing.assert_allclose(ev.cpu().numpy()[0], want, rtol=0, atol=1e-9)
