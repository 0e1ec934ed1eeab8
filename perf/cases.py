"""Workloads of the typed-graphlet library, each one pass through its public
entry points: one graph per call from a hundred edges to ten million, batches
of small graphs, a burst of served requests, and the calls that build on the
counts (position-aware and directed counts, the sparse form, embeddings).

``listed()`` names the fixed cases, ``draw(rng)`` gives others of the same
ranges.  ``prepare(case, seed)`` builds the device graph and the buffers a
program keeps (workspace, outputs, batch plan, server), ``run(state)`` is one
pass, ``work(case)`` the bytes such a pass cannot do without, and
``exact(case, seed)`` the results by plain enumeration where that is quick.
Graphs are drawn on the GPU from the seed alone.
"""

from __future__ import annotations

import math
import time

import numpy as np
import torch

import paper_2010_14058_amd as tg
from paper_2010_14058_amd import serve

DEV = "cuda"


# ------------------------------------------------------------------ cases

def listed() -> list[dict]:
    return [
        # the smallest served request, with its per-edge table: launches and
        # host round trips are all there is
        dict(name="tiny_m100", kind="count", shape="power", m=100, n=20, beta=2.2, wmax=12.0, L=6,
             rows=True),
        # the Erdos-Renyi configuration: n = 2000, average degree 8, L = 3
        dict(name="er_n2000", kind="count", shape="er", m=8000, n=2000, beta=0.0, wmax=0.0, L=3,
             rows=True),
        # a mid-size power law counted and then kept in the sparse form
        dict(name="sparse_m300k", kind="sparse", shape="power", m=300_000, n=30_000, beta=2.1,
             wmax=14722.0, L=5, rows=True),
        # the largest served request: global counts only
        dict(name="request_m1M", kind="count", shape="power", m=1_000_000, n=200_000, beta=2.2,
             wmax=2828.0, L=6, rows=False),
        # the power-law configuration: 1M nodes, 10M edges, per-edge table
        dict(name="power_m10M", kind="count", shape="power", m=10_000_000, n=1_000_000, beta=2.1,
             wmax=85000.0, L=5, rows=True),
        # the tripartite configuration at a quarter of its size: no triangles,
        # 4-cycles and long rows of few types
        dict(name="tripartite_m5M", kind="count", shape="tripartite", m=5_000_000, n=312_500,
             beta=2.3, wmax=25000.0, L=3, rows=True),
        # a service's small batch
        dict(name="batch_g1000", kind="batch", graphs=1000),
        # the batched configuration at half its size: global vectors of many
        # graphs of 10 to 500 nodes, each with its own number of types
        dict(name="batch_g50000", kind="batch", graphs=50_000),
        # position-aware counts of a power law with 1M edges
        dict(name="position_m1M", kind="position", shape="power", m=1_000_000, n=100_000, beta=2.1,
             wmax=26879.0, L=5, rows=True),
        # directed counts of the power-law configuration (a fifth reciprocal)
        dict(name="directed_m10M", kind="directed", shape="power", m=10_000_000, n=1_000_000,
             beta=2.1, wmax=85000.0, L=5, rows=True),
        # Alg. 5 for triangles of type 0: weights and a 16-dimensional
        # embedding of each component
        dict(name="embed_n20k", kind="embed", shape="power", m=200_000, n=20_000, beta=2.1,
             wmax=12020.0, L=5, graphlet=2, dim=16),
        # a burst of requests from host memory through the server, edges
        # log-uniform in 10^2..10^6
        dict(name="serve_burst48", kind="serve", requests=48, m_hi=1_000_000),
    ]


def _log_uniform(rng, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["count", "count", "count", "count", "count", "batch", "batch", "sparse",
                       "position", "directed", "embed", "serve"])
    if kind == "batch":
        return dict(kind="batch", graphs=_log_uniform(rng, 20, 50_000))
    if kind == "serve":
        return dict(kind="serve", requests=rng.randint(4, 64),
                    m_hi=_log_uniform(rng, 10_000, 1_000_000))
    if kind == "embed":
        n = _log_uniform(rng, 500, 25_000)
        return dict(kind="embed", shape="power", m=10 * n, n=n, beta=2.1,
                    wmax=round(85.0 * math.sqrt(n), 1), L=rng.choice([2, 3, 5]),
                    graphlet=rng.choice([1, 2]), dim=rng.choice([2, 8, 16]))
    L = rng.choice([1, 2, 3, 4, 5, 5, 6, 7, 8])
    # tables and scratch grow with L^2 per edge
    m_max = {"count": 2.4e8, "sparse": 2.5e7, "position": 3e7, "directed": 2.4e8}[kind] / (L * L)
    m = _log_uniform(rng, 100, min(m_max, 10_000_000))
    shape = rng.choice(["power", "power", "power", "er", "tripartite"]) if kind == "count" else "power"
    case = dict(kind=kind, shape=shape, m=m, beta=0.0, wmax=0.0, L=L, rows=True)
    if shape == "er":
        case["n"] = max(int(2 * math.sqrt(m)) + 2, int(m / rng.uniform(2.0, 20.0)))
    elif shape == "tripartite":
        case["m"] = m = min(m, 5_000_000)
        case["L"] = 3
        case["n"] = max(int(12 * math.sqrt(m)), m // 16)
        case["beta"] = 2.3
        case["wmax"] = round(11.0 * math.sqrt(m), 1)
    else:
        # the power-law configuration's hubs (25 sqrt(m)) down to the served
        # requests' (2 sqrt(2 m)), five or ten edges per node
        case["n"] = max(int(2 * math.sqrt(m)) + 2, m // rng.choice([5, 10]))
        case["beta"] = rng.choice([2.1, 2.2, 2.5])
        case["wmax"] = round(rng.choice([3.0, 9.0, 26.0]) * math.sqrt(m), 1)
    if kind == "count":
        case["rows"] = rng.random() < 0.7
    return case


# ----------------------------------------------------------------- graphs

class _Graph:
    """Device CSR (sorted rows, symmetric, simple) with node types, from the
    sorted keys lo * n + hi of its edges."""

    def __init__(self, n, key, types, L):
        lo = torch.div(key, n, rounding_mode="floor")
        hi = key - lo * n
        slots = torch.sort(torch.cat([key, hi * n + lo])).values
        src = torch.div(slots, n, rounding_mode="floor")
        self.col = (slots - src * n).to(torch.int32)
        self.row_ptr = torch.searchsorted(src, torch.arange(n + 1, device=DEV))
        self.src = src
        self.lo, self.hi = lo, hi          # canonical edges, lexicographic
        self.types = types.to(torch.uint8)
        self.n, self.m, self.L = n, int(lo.numel()), L


def _keys(n, u, v):
    lo, hi = torch.minimum(u, v), torch.maximum(u, v)
    keep = lo != hi
    return torch.unique(lo[keep] * n + hi[keep])


def _edges(gen, n, m, pairs):
    """Keys of exactly m distinct edges: pairs(k) draws k endpoint pairs;
    repeats are dropped and made up for (at last by uniform pairs), a surplus
    is dropped at random."""
    key = torch.empty(0, dtype=torch.int64, device=DEV)
    for turn in range(200):
        k = int(1.13 * (m - key.numel())) + 16
        if turn < 6:
            u, v = pairs(k)
        else:
            u, v = torch.randint(n, (2, k), generator=gen, device=DEV)
        key = torch.unique(torch.cat([key, _keys(n, u, v)]))
        if key.numel() >= m:
            break
    keep = torch.argsort(torch.rand(key.numel(), generator=gen, device=DEV))[:m]
    return torch.sort(key[keep]).values


def _pick(gen, cdf, k):
    x = torch.rand(k, generator=gen, device=DEV, dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, x, right=True).clamp_(max=cdf.numel() - 1)


def _power_weights(n, beta, mean, wmax):
    """w_v proportional to (v + v0)^(-1/(beta-1)), the largest about wmax
    (never below the mean), the mean as given."""
    a = 1.0 / (beta - 1.0)
    target = min(max(wmax / mean, 1.05), 0.5 * n)
    v = torch.arange(n, device=DEV, dtype=torch.float64)
    lo, hi = 1e-9, float(10 * n)
    for _ in range(40):
        mid = math.sqrt(lo * hi)
        w = (v + mid) ** (-a)
        if float(w[0] / w.mean()) > target:
            lo = mid
        else:
            hi = mid
    w = (v + math.sqrt(lo * hi)) ** (-a)
    return w * (mean / w.mean())


def _types(gen, n, L):
    """Node types with Zipf(1.2) frequencies."""
    p = torch.arange(1, L + 1, device=DEV, dtype=torch.float64) ** -1.2
    return _pick(gen, torch.cumsum(p, 0), n)


def _power(gen, case):
    """Chung-Lu power law, 60 % of the edges within a type."""
    n, m, L = case["n"], case["m"], case["L"]
    w = _power_weights(n, case["beta"], 2.0 * m / n, case["wmax"])
    types = _types(gen, n, L)
    cdf = torch.cumsum(w, 0)

    def pairs(k):
        u, v = _pick(gen, cdf, k), _pick(gen, cdf, k)
        same = torch.rand(k, generator=gen, device=DEV) < 0.4
        tu = types[u]
        for t in range(L):
            sel = torch.nonzero(same & (tu == t)).flatten()
            members = torch.nonzero(types == t).flatten()
            if sel.numel() and members.numel():
                v[sel] = members[_pick(gen, torch.cumsum(w[members], 0), sel.numel())]
        return u, v

    return _Graph(n, _edges(gen, n, m, pairs), types, L)


def _er(gen, case):
    n, m = case["n"], case["m"]
    key = _edges(gen, n, m, lambda k: torch.randint(n, (2, k), generator=gen, device=DEV))
    types = torch.randint(case["L"], (n,), generator=gen, device=DEV)
    return _Graph(n, key, types, case["L"])


def _tripartite(gen, case):
    """Classes A, B, C of 80, 16 and 4 % of the nodes; half of the edges join
    A and B, 30 % A and C, 20 % B and C; B and C endpoints by power-law weight."""
    n, m = case["n"], case["m"]
    nB, nC = max(4, n * 16 // 100), max(4, n * 4 // 100)
    nA = n - nB - nC
    mAB, mAC, mBC = m // 2, (3 * m) // 10, m // 5   # of the wanted edges
    wB = _power_weights(nB, case["beta"], (mAB + mBC) / nB, case["wmax"])
    wC = _power_weights(nC, case["beta"], (mAC + mBC) / nC, case["wmax"])
    cB, cC = torch.cumsum(wB, 0), torch.cumsum(wC, 0)

    def pairs(k):
        kAB, kAC, kBC = k // 2, (3 * k) // 10, k // 5 + 1
        a = torch.randint(nA, (kAB + kAC,), generator=gen, device=DEV)
        b = nA + _pick(gen, cB, kAB + kBC)
        c = nA + nB + _pick(gen, cC, kAC + kBC)
        return torch.cat([a, b[kAB:]]), torch.cat([b[:kAB], c])

    types = torch.zeros(n, device=DEV, dtype=torch.int64)
    types[nA:nA + nB] = 1
    types[nA + nB:] = 2
    return _Graph(n, _edges(gen, n, m, pairs), types, 3)


def _graph(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return {"power": _power, "er": _er, "tripartite": _tripartite}[case["shape"]](gen, case)


def _shuffled(g, seed):
    """The same graph under a random numbering of its nodes."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    p = torch.argsort(torch.rand(g.n, generator=gen, device=DEV))
    types = torch.empty_like(g.types)
    types[p] = g.types
    return _Graph(g.n, _keys(g.n, p[g.lo], p[g.hi]), types, g.L)


def _batch(graphs, seed):
    """Small Chung-Lu graphs as one disjoint union: 10 to 500 nodes
    (lognormal), average degree 4 to 12, 4 to 8 uniform types each."""
    rng = np.random.default_rng(seed)
    n = np.clip(np.round(np.exp(rng.normal(4.0, 1.0, graphs))), 10, 500).astype(np.int64)
    dbar = rng.uniform(4.0, 12.0, graphs)
    L = rng.permutation(4 + np.arange(graphs) % 5).astype(np.int32)
    node_ptr = np.concatenate([[0], np.cumsum(n)])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    N = int(node_ptr[-1])
    n_d, d_d = torch.from_numpy(n).to(DEV), torch.from_numpy(dbar).to(DEV)
    ptr = torch.from_numpy(node_ptr).to(DEV)
    gid = torch.repeat_interleave(torch.arange(graphs, device=DEV), n_d)
    w = (torch.arange(N, device=DEV) - ptr[gid] + 1).to(torch.float64) ** (-1.0 / 1.5)
    total = torch.zeros(graphs, device=DEV, dtype=torch.float64)
    total = torch.cumsum(w, 0)[ptr[1:] - 1].diff(prepend=total[:1])
    w = torch.minimum(w * (d_d * n_d / total)[gid], (2.0 * torch.sqrt(n_d * d_d))[gid])
    cdf = torch.cumsum(w, 0)
    end = cdf[ptr[1:] - 1]
    start = torch.cat([end.new_zeros(1), end[:-1]])
    draws = torch.round(n_d * d_d / 2).to(torch.int64)
    eg = torch.repeat_interleave(torch.arange(graphs, device=DEV), draws)

    def ends():
        x = start[eg] + torch.rand(eg.numel(), generator=gen, device=DEV,
                                   dtype=torch.float64) * (end - start)[eg]
        v = torch.searchsorted(cdf, x, right=True)
        return torch.minimum(torch.maximum(v, ptr[eg]), ptr[eg + 1] - 1)

    L_d = torch.from_numpy(L.astype(np.int64)).to(DEV)
    types = torch.floor(torch.rand(N, generator=gen, device=DEV) * L_d[gid])
    types = torch.minimum(types.to(torch.int64), L_d[gid] - 1)
    g = _Graph(N, _keys(N, ends(), ends()), types, int(L.max()))
    return g, node_ptr, L


def _requests(case, seed):
    """Host arrays of the burst's graphs: edges log-uniform from 100 to m_hi,
    five edges per node, exponent 2.2, six types."""
    rng = np.random.default_rng(seed)
    out = []
    for r in range(case["requests"]):
        m = int(round(math.exp(rng.uniform(math.log(100), math.log(case["m_hi"])))))
        n = max(20, m // 5)
        g = _graph(dict(shape="power", n=n, m=m, L=6, beta=2.2,
                        wmax=round(2.0 * math.sqrt(2.0 * m), 1)), seed * 1009 + r)
        out.append((g.row_ptr.cpu().numpy(), g.col.cpu().numpy(), g.types.cpu().numpy()))
    return out


# ------------------------------------------------------------------ states

class _State:
    def __init__(self, kind):
        self.kind = kind
        self.server = None

    def __del__(self):
        if self.server is not None:
            self.server.close()


def prepare(case: dict, seed: int) -> _State:
    s = _State(case["kind"])
    if s.kind == "batch":
        g, node_ptr, L = _batch(case["graphs"], seed)
        s.plan = tg.BatchPlan(g.row_ptr, g.col, g.types, node_ptr, L)
        s.out = torch.empty(int(s.plan.goff_host[-1]), dtype=torch.int64, device=DEV)
        s.ws = tg.Workspace(DEV)
        s.ws.get(tg.batch_workspace_bytes(s.plan.n, s.plan.nnz, s.plan.G, s.plan.L_max))
        return s
    if s.kind == "serve":
        s.graphs = _requests(case, seed)
        s.server = serve.Server(40 << 30, workers=2, worker_bytes=16 << 30)
        return s
    if s.kind == "sparse":
        # one graph, its nodes numbered by the seed: the number of nonzero
        # counts stays the same
        g = _shuffled(_graph(case, 1), seed)
    else:
        g = _graph(case, seed)
    s.rp, s.col, s.types, s.L = g.row_ptr, g.col, g.types, g.L
    s.ws = tg.Workspace(DEV)
    if s.kind == "embed":
        s.graphlet, s.dim = case["graphlet"], case["dim"]
        s.rows, _ = tg.count_typed_graphlets(s.rp, s.col, s.types, s.L)
        s.uv = tg.edge_list(s.rp, s.col)
        s.multiset = _multiset(case)
    elif s.kind == "directed":
        # a fifth of the edges reciprocal, else one arc of a fair direction
        gen = torch.Generator(device=DEV)
        gen.manual_seed(seed + 1)
        r = torch.rand(g.m, generator=gen, device=DEV)
        code = torch.where(r < 0.2, 3, torch.where(r < 0.6, 1, 2))
        src, dst = g.src, g.col.long()
        eid = torch.searchsorted(g.lo * g.n + g.hi,
                                 torch.minimum(src, dst) * g.n + torch.maximum(src, dst))
        c = code[eid]
        s.dirs = torch.where(src < dst, c, ((c & 1) << 1) | (c >> 1)).to(torch.uint8)
    else:
        s.ws.get(tg.workspace_bytes(g.n, 2 * g.m, g.L))
        pa = s.kind == "position"
        width = tg.pa_row_width(g.L) if pa else tg.row_width(g.L)
        gw = tg.pa_global_width(g.L) if pa else tg.global_width(g.L)
        s.per_edge = case["rows"]
        s.rows = torch.empty((g.m, width), dtype=torch.int64, device=DEV) if s.per_edge else None
        s.glob = torch.empty(gw, dtype=torch.int64, device=DEV)
    return s


def _multiset(case):
    # triangles of type 0; 3-paths of types 0, 0 and 1
    return [0, 0, 0] if case["graphlet"] == 2 else [0, 0, 1]


def run(s: _State):
    if s.kind == "batch":
        glob, _ = tg.count_batch(s.plan, out_globals=s.out, workspace=s.ws)
        return {"globals": glob}
    if s.kind == "serve":
        reqs = [serve.Request(rid=k, row_ptr=rp, col=col, types=ty, L=6)
                for k, (rp, col, ty) in enumerate(s.graphs)]
        done = len(s.server.done) + len(reqs)
        for r in reqs:
            s.server.submit(r)
        while len(s.server.done) < done:
            time.sleep(1e-4)
        return {"status": np.array([r.status for r in reqs]),
                "globals": np.concatenate([r.result for r in reqs]).view(np.int64)}
    if s.kind == "embed":
        w = tg.graphlet_weights(s.rows, s.uv, s.types, s.L, s.graphlet, s.multiset)
        Z, ev, comp, _ = tg.graphlet_embedding(s.rp, s.col, w, s.dim, workspace=s.ws)
        return {"weights": w, "Z": Z, "eigenvalues": ev, "component": comp}
    if s.kind == "directed":
        rows, glob = tg.count_directed(s.rp, s.col, s.dirs, s.types, s.L, workspace=s.ws)
        return {"rows": rows, "globals": glob}
    count = tg.count_position_aware if s.kind == "position" else tg.count_typed_graphlets
    rows, glob = count(s.rp, s.col, s.types, s.L, per_edge=s.per_edge, out_rows=s.rows,
                       out_global=s.glob, workspace=s.ws)
    out = {"globals": glob}
    if rows is not None:
        out["rows"] = rows
    if s.kind == "sparse":
        off, keys, counts = tg.sparse_rows(rows, s.L, workspace=s.ws)
        out.update(offsets=off, keys=keys, counts=counts)
    return out


# -------------------------------------------------------------------- work

def work(case: dict) -> dict:
    """Inputs read once and outputs written once (nominal sizes)."""
    kind = case["kind"]
    if kind == "batch":
        # 87 nodes and 300 edges per graph on average; 1,130 global counts
        return {"bytes": case["graphs"] * (87 * 9 + 600 * 4 + 1130 * 8.0), "flops": 0}
    if kind == "serve":
        mean = (case["m_hi"] - 100) / math.log(case["m_hi"] / 100)
        return {"bytes": case["requests"] * (mean * 8 + mean / 5 * 9 + 1050 * 8.0), "flops": 0}
    n, m, L = case["n"], case["m"], case["L"]
    graph = 8.0 * (n + 1) + 8.0 * m + n
    if kind == "embed":
        # the completing columns of each row, the edge list, weights, Z and
        # the spectra
        return {"bytes": graph + m * (8.0 + 16 + 16) + 16.0 * n * case["dim"], "flops": 0}
    if kind == "directed":
        return {"bytes": graph + 2.0 * m + 8.0 * (m * 15 * L + 4 * L * L + 64 * L ** 3), "flops": 0}
    P = L * (L + 1) // 2
    if kind == "position":
        return {"bytes": graph + 8.0 * m * (3 * L + 10 * L * L + 5 * P), "flops": 0}
    table = 8.0 * m * (2 * L + 10 * P) if case["rows"] else 0.0
    out = table
    if kind == "sparse":
        out += table + 0.6 * table * 10 / 8 + 8.0 * m     # read again, entries and offsets
    return {"bytes": graph + out, "flops": 0}


# ------------------------------------------------------------------- exact

def _rank(multiset) -> int:
    """Co-lexicographic rank of a type multiset."""
    return sum(math.comb(t + q, q + 1) for q, t in enumerate(sorted(multiset)))


def _exact_rows(n, src, col, u, v, types, L):
    """Every edge's typed counts: the classes of the other nodes by their
    adjacency to the edge's ends, and the adjacent pairs between classes."""
    A = np.zeros((n, n), dtype=np.int64)
    A[src, col] = 1
    onehot = np.eye(L, dtype=np.int64)[types]
    tdeg = A @ onehot
    P = [(t, w) for t in range(L) for w in range(t, L)]
    rows = np.zeros((u.shape[0], 2 * L + 10 * len(P)), dtype=np.int64)
    for e, (i, j) in enumerate(zip(u, v)):
        near = A[i] + 2 * A[j]
        near[i] = near[j] = 0
        K = np.flatnonzero(near)
        cls = (near[K] - 1) * L + types[K]
        H = np.zeros((K.shape[0], 3 * L), dtype=np.int64)
        H[np.arange(K.shape[0]), cls] = 1
        cnt = H.sum(0)
        sub = A[np.ix_(K, K)]
        M = H.T @ sub @ H
        far = tdeg[K] - sub @ onehot[K]
        far[:, types[i]] -= A[K, i]
        far[:, types[j]] -= A[K, j]
        far = H.T @ far                       # pairs with a node next to neither end
        I, J, T = (slice(q * L, (q + 1) * L) for q in range(3))
        rows[e, :L] = cnt[T]
        rows[e, L:2 * L] = cnt[I] + cnt[J]

        def within(S):                        # unordered pairs of one class: (adjacent, all)
            a = M[S, S]
            c = np.outer(cnt[S], cnt[S])
            d = np.diag_indices(L)
            a2, c2 = a.copy(), c.copy()
            a2[d] = a[d] // 2
            c2[d] = cnt[S] * (cnt[S] - 1) // 2
            return a2, c2

        def across(S, R):                     # pairs of two classes, by type pair
            a, c = M[S, R], np.outer(cnt[S], cnt[R])
            return fold(a), fold(c)

        def fold(a):
            b = a + a.T
            d = np.diag_indices(L)
            b[d] = a[d]
            return b

        ii, jj, tt = within(I), within(J), within(T)
        ij, ti, tj = across(I, J), across(T, I), across(T, J)
        blocks = [fold(far[I] + far[J]), ij[1] - ij[0], ii[1] - ii[0] + jj[1] - jj[0], ij[0],
                  ii[0] + jj[0], fold(far[T]), ti[1] - ti[0] + tj[1] - tj[0], ti[0] + tj[0],
                  tt[1] - tt[0], tt[0]]
        for b, a in enumerate(blocks):
            rows[e, 2 * L + b * len(P):2 * L + (b + 1) * len(P)] = [a[t, w] for t, w in P]
    return rows


def _exact_globals(rows, u, v, types, L):
    P = [(t, w) for t in range(L) for w in range(t, L)]
    sizes = [math.comb(L + 1, 2)] + 2 * [math.comb(L + 2, 3)] + 6 * [math.comb(L + 3, 4)]
    start = np.concatenate([[0], np.cumsum(sizes)])
    glob = np.zeros(start[-1], dtype=np.int64)
    graphlet = [3, 3, 4, 5, 6, 6, 6, 7, 7, 8]          # of orbits g3..g12
    a, b = types[u].astype(int), types[v].astype(int)
    for x in range(L):
        for y in range(x, L):
            sel = (np.minimum(a, b) == x) & (np.maximum(a, b) == y)
            tot = rows[sel].sum(0)
            glob[_rank((x, y))] = sel.sum()
            for t in range(L):
                glob[start[2] + _rank((x, y, t))] += tot[t]
                glob[start[1] + _rank((x, y, t))] += tot[L + t]
            for o in range(10):
                for p, (t, w) in enumerate(P):
                    glob[start[graphlet[o]] + _rank((x, y, t, w))] += tot[2 * L + o * len(P) + p]
    for h, edges in enumerate([1, 2, 3, 3, 3, 4, 4, 5, 6]):
        glob[start[h]:start[h + 1]] //= edges
    return glob


def _exact_embedding(case, n, src, col, u, v, types):
    """Instance weights of the graphlet and, per component of the weighted
    graph, the smallest eigenvalues of its normalised Laplacian."""
    A = np.zeros((n, n))
    A[src, col] = 1
    want = sorted(_multiset(case))
    w = np.zeros(u.shape[0])
    for e, (i, j) in enumerate(zip(u, v)):
        rest = list(want)
        try:
            rest.remove(types[i])
            rest.remove(types[j])
        except ValueError:
            continue
        third = A[i] * A[j] if case["graphlet"] == 2 else np.abs(A[i] - A[j])
        third[i] = third[j] = 0
        w[e] = third[types == rest[0]].sum()
    W = np.zeros((n, n))
    W[u, v] = w
    W[v, u] = w
    comp = np.where(W.any(1), np.arange(n), -1)
    while True:
        near = np.where(W > 0, np.where(comp >= 0, comp, n)[None, :], n).min(1)
        new = np.where(comp >= 0, np.minimum(comp, near), -1)
        if (new == comp).all():
            break
        comp = new
    ev = np.zeros((n, case["dim"]))
    for r in np.unique(comp[comp >= 0]):
        nodes = np.flatnonzero(comp == r)
        sub = W[np.ix_(nodes, nodes)]
        d = 1.0 / np.sqrt(sub.sum(1))
        lam = np.linalg.eigvalsh(np.eye(nodes.size) - d[:, None] * sub * d[None, :])
        k = min(case["dim"], nodes.size)
        ev[r, :k] = lam[:k]
    return {"weights": w.astype(np.int64), "Z": None, "eigenvalues": ev, "component": comp}


def exact(case: dict, seed: int):
    kind = case["kind"]
    if kind not in ("count", "embed") or case["n"] > 2500 or case["m"] > 25_000:
        return None
    g = _graph(case, seed)
    src, col = g.src.cpu().numpy(), g.col.cpu().numpy()
    u, v, types = g.lo.cpu().numpy(), g.hi.cpu().numpy(), g.types.cpu().numpy()
    if kind == "embed":
        return _exact_embedding(case, g.n, src, col, u, v, types)
    if case["m"] > 10_000:
        return None
    rows = _exact_rows(g.n, src, col, u, v, types, g.L)
    out = {"globals": _exact_globals(rows, u, v, types, g.L)}
    if case["rows"]:
        out["rows"] = rows
    return out
