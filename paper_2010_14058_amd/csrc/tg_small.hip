// Global typed counts of batches of small graphs (at most SMALL_NODES nodes
// each, no per-edge table): one workgroup per graph, the whole graph in LDS
// as an adjacency bit matrix.
//
// The global vector needs no per-edge orbit counts.  For every type multiset
// the instances of the six connected 4-node graphlets follow from the numbers
// of not necessarily induced copies on node sets of that multiset (a spanning
// subgraph keeps the node set, so the untyped relations hold per multiset):
//   K4 = h8                              cliques
//   DIA = h7 + 6 h8                      two triangles on an edge
//   TAIL = h6 + 4 h7 + 12 h8             a triangle and an edge at a corner
//   C4 = h5 + h7 + 3 h8                  cycles
//   STAR = h4 + h6 + 2 h7 + 4 h8         three neighbours of a node
//   P4 = h3 + 4 h5 + 2 h6 + 6 h7 + 12 h8 paths
// and for 3 nodes P3 = h1 + 3 h2.  STAR and P3 are sums over nodes of products
// of typed degrees, P4, TAIL and DIA sums over edges of products of typed
// degrees and typed triangle counts, C4 a sum over node pairs of products of
// typed common-neighbour counts, and K4 bit-matrix intersections.  Nodes are
// ranked by degree, so that a cycle taken once, at its highest-ranked node,
// and a clique taken from its highest-ranked edge meet few candidates.
#include <hip/hip_runtime.h>

#include "tg_device.hpp"

namespace tg {

constexpr int SMALL_THREADS = 256;          // threads of the check kernel
// Threads per workgroup by size class, for batches that fill the chip several
// times over and for those of at most SMALL_FEW graphs per CU, where the time
// of one graph counts: 50,000 graphs take 1.29 + 1.07 ms (128 and 256 nodes)
// with the first and 1.87 + 1.31 ms with the second, 1,000 graphs 148 + 188 us
// and 101 + 128 us.
constexpr int SMALL_NT_LO = 256, SMALL_NT_MID = 512, SMALL_NT_HI = 1024;
constexpr int SMALL_FEW = 4;

// Layout of the workgroup's LDS, in bytes from its base, for graphs of at most
// `nodes` nodes and L types.  Sums of copies stay below 24 C(nodes, 4) (at most
// 12 paths on four nodes; tailed triangles are met twice), so graphs of at
// most 256 nodes need only 32-bit sums.
static_assert((uint64_t)SMALL_MID * (SMALL_MID - 1) * (SMALL_MID - 2) * (SMALL_MID - 3) <= 0xffffffffu,
              "sums of copies of graphs of SMALL_MID nodes in 32 bits");
struct SmallLds {
    size_t hist, bits, masks, rank4, rank3, pairs, triples, cnt, pair, scan, deg, row, rank, types, total;
};

__host__ __device__ inline int small_c3(int L) { return L * (L + 1) * (L + 2) / 6; }
__host__ __device__ inline int small_c4(int L) {
    return L * (L + 1) / 2 * (L + 2) / 3 * (L + 3) / 4;
}
__host__ __device__ inline int small_pairs(int L) { return L * (L + 1) / 2; }

// 64-bit words of a bit row (1, 2, 4 or 8: one instance of the pair kernels
// each, so that a row stays in registers) and their pitch: odd, so that the
// same word of consecutive rows falls into different LDS banks.
__host__ __device__ inline int small_words(int nodes) {
    return nodes <= 64 ? 1 : nodes <= 128 ? 2 : nodes <= 256 ? 4 : 8;
}
__host__ __device__ inline int small_stride(int nodes) { return small_words(nodes) | 1; }

__host__ __device__ inline SmallLds small_lds(int nodes, int L, int threads) {
    const int P = small_pairs(L);
    SmallLds y{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = (o + bytes + 15) & ~size_t(15);
        return at;
    };
    y.hist = take((nodes <= SMALL_MID ? sizeof(uint32_t) : sizeof(uint64_t)) * (size_t)(P + 2 * small_c3(L) + 6 * small_c4(L)));
    y.bits = take(sizeof(uint64_t) * (size_t)nodes * small_stride(nodes));
    y.masks = take(sizeof(uint64_t) * (size_t)L * small_words(nodes));
    y.rank4 = take(sizeof(uint16_t) * (size_t)P * P);
    y.rank3 = take(sizeof(uint16_t) * (size_t)P * L);
    y.pairs = take(sizeof(uint16_t) * (size_t)P);
    y.triples = take(sizeof(uint16_t) * (size_t)small_c3(L));
    y.pair = take(sizeof(uint32_t) * 4 * (size_t)threads);   // two queues per wave
    y.scan = take(sizeof(uint32_t) * (size_t)threads);
    y.deg = take(sizeof(uint16_t) * (size_t)nodes * L);
    y.types = take((size_t)nodes);
    // row offsets and ranks are needed until the bit matrix stands, the
    // counts of queued pairs after it
    const size_t rows = sizeof(uint32_t) * (size_t)(nodes + 1);
    const size_t cnts = sizeof(uint16_t) * (size_t)threads * L;
    const size_t load = rows + sizeof(uint16_t) * (size_t)nodes;
    y.cnt = y.row = take(cnts > load ? cnts : load);
    y.rank = y.row + rows;
    y.total = o;
    return y;
}

// Row of slot s (relative to the graph's first slot) among the n rows.
__device__ __forceinline__ int small_row(const uint32_t *row, int n, uint32_t s) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (row[mid + 1] <= s) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Input checks of every graph (the batch descriptor has passed its own):
// rows, types, and the symmetry of the adjacency from its bit matrix.  Only row
// offsets out of order stop a graph's other checks, and no graph those of
// another, so that the status code knows every error.
__global__ void __launch_bounds__(SMALL_THREADS)
k_small_check(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
              const uint8_t *__restrict__ types, const int64_t *__restrict__ node_ptr,
              const int32_t *__restrict__ gL, const uint32_t *__restrict__ list, int step,
              const uint64_t *__restrict__ counters, int c_count, int max_nodes, int64_t n_all,
              int64_t nnz, uint32_t *__restrict__ status) {
    extern __shared__ unsigned long long sm_check[];
    if (failed_before(status, ST_INPUT & ~ST_BATCH)) return;
    unsigned long long *bits = sm_check;
    uint32_t *row = reinterpret_cast<uint32_t *>(bits + (size_t)max_nodes * small_stride(max_nodes));
    const int tid = threadIdx.x;
    const uint64_t count = counters[c_count];
    for (uint64_t at = blockIdx.x; at < count; at += gridDim.x) {
        const int64_t g = list[(int64_t)step * (int64_t)at];
        const int64_t a = node_ptr[g];
        const int n = (int)(node_ptr[g + 1] - a);
        if (n <= 0) continue;
        const int stride = small_stride(n);
        uint32_t bad = 0;
        const int64_t s0 = rp[a];
        for (int v = tid; v <= n; v += SMALL_THREADS) {
            const int64_t e = rp[a + v];
            // offsets from the graph's first slot; a graph of n nodes has
            // fewer than n^2 slots
            const int64_t o = e - s0;
            if (s0 < 0 || o < 0 || e > nnz || o > (int64_t)n * n) bad |= ST_ROW_BOUNDS;
            row[v] = (uint32_t)o;
            if (v < n) {
                if (rp[a + v + 1] < e) bad |= ST_ROW_BOUNDS;
                if (types[a + v] >= gL[g]) bad |= ST_TYPE_RANGE;
            }
        }
        if (tid == 0 && ((a == 0 && s0 != 0) || (a + n == n_all && rp[n_all] != nnz)))
            bad |= ST_ROW_BOUNDS;
        for (int q = tid; q < n * stride; q += SMALL_THREADS) bits[q] = 0ull;
        if (__syncthreads_or((bad & ST_ROW_BOUNDS) != 0)) {
            if (bad) atomicOr(status, bad);
            continue;
        }
        const uint32_t slots = row[n];
        for (uint32_t s = tid; s < slots; s += SMALL_THREADS) {
            const int u = small_row(row, n, s);
            const int64_t x = col[s0 + s];
            if (x < 0 || x >= n_all) bad |= ST_COL_RANGE;
            else if (x < a || x >= a + n) bad |= ST_CROSS_GRAPH;
            else atomicOr(&bits[u * stride + (int)((x - a) >> 6)], 1ull << ((x - a) & 63));
            if (x == a + u) bad |= ST_SELF_LOOP;
            if (s > row[u] && col[s0 + s - 1] >= x) bad |= ST_UNSORTED;
        }
        if (!__syncthreads_or(bad != 0)) {
            for (uint32_t s = tid; s < slots; s += SMALL_THREADS) {
                const int u = small_row(row, n, s);
                const int x = (int)(col[s0 + s] - a);
                if (!((bits[x * stride + (u >> 6)] >> (u & 63)) & 1ull)) bad |= ST_ASYMMETRIC;
            }
        }
        if (bad) atomicOr(status, bad);
        __syncthreads();
    }
}

// Views of one graph in LDS.  HT: word of the sums.
template <typename HT>
struct SmallGraph {
    int n, stride, L, P;
    unsigned long long *bits;
    const uint64_t *masks;     // [L][W] nodes of each type
    const uint16_t *rank4, *rank3, *pairs;
    uint16_t *deg;
    const uint8_t *types;
    int pmax;                  // row length of the rank tables
    int lmax;
    HT *h0, *p3, *k3, *k4, *dia, *tail, *c4, *star, *p4;
};

__device__ __forceinline__ int small_rank2(int a, int b) {
    return a <= b ? a + b * (b + 1) / 2 : b + a * (a + 1) / 2;
}

__device__ __forceinline__ void small_add(uint32_t *p, uint32_t v) {
    if (v) atomicAdd(p, v);
}
__device__ __forceinline__ void small_add(unsigned long long *p, unsigned long long v) {
    if (v) atomicAdd(p, v);
}

// Typed counts of the bits x[0..W) of each lane, one type at a time (uniform
// over the wave, so the mask reads are broadcasts and overlap).
template <int W, typename HT>
__device__ __forceinline__ void small_typed(const SmallGraph<HT> &G, const unsigned long long (&x)[W],
                                            uint16_t *c) {
    for (int t = 0; t < G.L; ++t) {
        int k = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) k += __popcll(x[q] & G.masks[t * W + q]);
        c[t] = (uint16_t)k;
    }
}

// The edges of `have` <= 64 queued pairs v > w (ranks) of one wave.  Typed
// triangle counts, one edge per lane; cliques, one triangle per lane and step
// (a hub edge's triangles are spread over the wave); then one (edge, type
// pair) per lane and step, each lane keeping its type pair.
template <int W, typename HT>
__device__ void small_edges(const SmallGraph<HT> &G, const uint32_t *pair, uint16_t *cnt,
                            uint32_t *scan, int have) {
    const int lane = lane_id();
    const int L = G.L, P = G.P;
    uint32_t below = 0;   // triangles with a third node below w
    if (lane < have) {
        const int v = pair[lane] & 1023, w = pair[lane] >> 10;
        const unsigned long long *rv = G.bits + v * G.stride, *rw = G.bits + w * G.stride;
        atomicAdd(&G.h0[small_rank2(G.types[v], G.types[w])], (HT)1);
        unsigned long long x[W];
#pragma unroll
        for (int q = 0; q < W; ++q) x[q] = rv[q] & rw[q];
        small_typed<W>(G, x, cnt + lane * L);
#pragma unroll
        for (int q = 0; q < W; ++q) {
            if (q < (w >> 6)) below += (uint32_t)__popcll(x[q]);
            else if (q == (w >> 6)) below += (uint32_t)__popcll(x[q] & ((1ull << (w & 63)) - 1ull));
        }
    }
    const uint32_t incl = wave_incl_scan(below);
    scan[lane] = incl;
    const uint32_t total = __shfl(incl, WAVE - 1, WAVE);
    wave_sync();
    for (uint32_t f = lane; f < total; f += WAVE) {
        const int o = owner_of(scan, WAVE, f);
        uint32_t r = f - (o ? scan[o - 1] : 0u);
        const int v = pair[o] & 1023, w = pair[o] >> 10;
        const unsigned long long *rv = G.bits + v * G.stride, *rw = G.bits + w * G.stride;
        // the r-th common neighbour k below w, then l < k adjacent to all
        int q = 0;
        unsigned long long m = rv[0] & rw[0];
        while (W > 1 && r >= (uint32_t)__popcll(m)) {
            r -= (uint32_t)__popcll(m);
            ++q;
            m = rv[q] & rw[q];
        }
        for (; r > 0; --r) m &= m - 1;
        const int b = __ffsll((long long)m) - 1;
        const int k = q * 64 + b;
        const unsigned long long *rk = G.bits + k * G.stride;
        const uint16_t *r4 = G.rank4 + small_rank2(G.types[v], G.types[k]) * G.pmax;
        const int tw = G.types[w];
        for (int z = 0; z <= q; ++z) {
            unsigned long long l = rv[z] & rw[z] & rk[z];
            if (z == q) l &= (1ull << b) - 1ull;
            for (int t = 0; l && t < L; ++t) {
                const unsigned long long y = l & G.masks[t * W + z];
                if (!y) continue;
                l ^= y;
                atomicAdd(&G.k4[r4[small_rank2(tw, t)]], (HT)__popcll(y));
            }
        }
    }
    // 64 / P edges per step, or more steps per edge for P > 64.  Lane e holds
    // edge e's ends and types, handed over by a shuffle, so that a step's table
    // reads do not wait for one another
    uint32_t mine = 0;
    if (lane < have)
        mine = pair[lane] | ((uint32_t)G.types[pair[lane] & 1023] << 20) |
               ((uint32_t)G.types[pair[lane] >> 10] << 24);
    const int per = P <= WAVE ? WAVE / P : 1;
    for (int p0 = 0; p0 < P; p0 += WAVE) {
        const int sub = P <= WAVE ? lane / P : 0;
        const int p = P <= WAVE ? lane - sub * P : p0 + lane;
        const bool on = sub < per && p < P;
        const int tu = on ? G.pairs[p] : 0;
        const int t = tu & 255, u = tu >> 8;
        const bool same = t == u;
        auto step = [&](uint32_t pr, int e) {
            const int v = pr & 1023, w = (pr >> 10) & 1023;
            const int a = (pr >> 20) & 15, b = pr >> 24;
            const uint16_t *dv = G.deg + v * L, *dw = G.deg + w * L, *c = cnt + e * L;
            const int ct = c[t], cu = c[u];
            const int ab = small_rank2(a, b);
            const int r = G.rank4[ab * G.pmax + p];
            // degrees without the edge itself
            const int vt = (int)dv[t] - (t == b), vu = (int)dv[u] - (u == b);
            const int wt = (int)dw[t] - (t == a), wu = (int)dw[u] - (u == a);
            // all below 2^20
            small_add(&G.p4[r], (HT)(same ? vt * wt - ct : vt * wu + vu * wt));
            if (!(ct | cu)) return;
            small_add(&G.dia[r], (HT)(same ? ct * (ct - 1) / 2 : ct * cu));
            small_add(&G.tail[r], (HT)(same ? ct * (vt + wt - 2) : ct * (vu + wu) + cu * (vt + wt)));
            if (same) small_add(&G.k3[G.rank3[ab * G.lmax + t]], (HT)ct);
        };
        if (per == 1) {
            // one edge per step: its ends and types in scalar registers
            for (int e = 0; e < have; ++e) {
                const uint32_t pr = (uint32_t)__builtin_amdgcn_readlane((int)mine, e);
                if (on) step(pr, e);
            }
        } else {
            for (int e0 = 0; e0 < have; e0 += per) {
                const int e = e0 + sub;
                const uint32_t pr = (uint32_t)__shfl((int)mine, e < have ? e : 0, WAVE);
                if (on && e < have) step(pr, e);
            }
        }
    }
    wave_sync();
}

// The 4-cycles of `have` <= 64 queued pairs v > w of one wave, v the highest
// rank of the cycle: products of the typed counts of their common neighbours
// below v, one pair per lane (few types are present in one pair).
template <int W, typename HT>
__device__ void small_cycles(const SmallGraph<HT> &G, const uint32_t *pair, uint16_t *cnt,
                             int have) {
    const int lane = lane_id();
    const int L = G.L;
    if (lane < have) {
        const int v = pair[lane] & 1023, w = pair[lane] >> 10;
        const unsigned long long *rv = G.bits + v * G.stride, *rw = G.bits + w * G.stride;
        uint16_t *c = cnt + lane * L;
        unsigned long long x[W];
#pragma unroll
        for (int q = 0; q < W; ++q) {
            x[q] = rv[q] & rw[q];
            if (q > (v >> 6)) x[q] = 0ull;
            else if (q == (v >> 6)) x[q] &= (1ull << (v & 63)) - 1ull;
        }
        small_typed<W>(G, x, c);
        const uint16_t *r4 = G.rank4 + small_rank2(G.types[v], G.types[w]) * G.pmax;
        for (int u = 0; u < L; ++u) {
            const uint32_t cu = c[u];
            if (!cu) continue;
            for (int t = 0; t < u; ++t)
                small_add(&G.c4[r4[t + u * (u + 1) / 2]], (HT)(c[t] * cu));
            small_add(&G.c4[r4[u + u * (u + 1) / 2]], (HT)(cu * (cu - 1) / 2));
        }
    }
    wave_sync();
}

// Takes 64 queued pairs away once they have been processed.
__device__ __forceinline__ void small_shift(uint32_t *queue, int have) {
    const int lane = lane_id();
    const uint32_t move = lane < have ? queue[WAVE + lane] : 0u;
    wave_sync();
    if (lane < have) queue[lane] = move;
    wave_sync();
}

// Every pair w < v of ranks, one row per wave: edges, and pairs with at least
// two common neighbours below v, each queued and taken 64 at a time.
template <int W, int NT, typename HT>
__device__ void small_all_pairs(const SmallGraph<HT> &G, uint32_t *equeue, uint32_t *cqueue,
                                uint16_t *cnt, uint32_t *scan) {
    const int lane = lane_id();
    int ne = 0, nc = 0;
    for (int v = G.n - 1 - (int)threadIdx.x / WAVE; v > 0; v -= NT / WAVE) {
        const unsigned long long *rv = G.bits + v * G.stride;
        unsigned long long xv[W];
#pragma unroll
        for (int q = 0; q < W; ++q) {
            xv[q] = q <= (v >> 6) ? rv[q] : 0ull;
            if (q == (v >> 6)) xv[q] &= (1ull << (v & 63)) - 1ull;
        }
        for (int w0 = 0; w0 < v; w0 += WAVE) {
            const int w = w0 + lane;
            bool edge = false, cyc = false;
            if (w < v) {
                const unsigned long long *rw = G.bits + w * G.stride;
                int c = 0;
#pragma unroll
                for (int q = 0; q < W; ++q) c += __popcll(xv[q] & rw[q]);
                edge = (rv[w >> 6] >> (w & 63)) & 1ull;
                cyc = c >= 2;
            }
            const uint32_t pr = (uint32_t)v | ((uint32_t)w << 10);
            const uint64_t before = (1ull << lane) - 1ull;
            const uint64_t be = __ballot(edge), bc = __ballot(cyc);
            if (!(be | bc)) continue;
            if (edge) equeue[ne + __popcll(be & before)] = pr;
            if (cyc) cqueue[nc + __popcll(bc & before)] = pr;
            ne += __popcll(be);
            nc += __popcll(bc);
            wave_sync();
            if (ne >= WAVE) {
                small_edges<W>(G, equeue, cnt, scan, WAVE);
                ne -= WAVE;
                small_shift(equeue, ne);
            }
            if (nc >= WAVE) {
                small_cycles<W>(G, cqueue, cnt, WAVE);
                nc -= WAVE;
                small_shift(cqueue, nc);
            }
        }
    }
    if (ne > 0) small_edges<W>(G, equeue, cnt, scan, ne);
    if (nc > 0) small_cycles<W>(G, cqueue, cnt, nc);
}

// One workgroup per graph at a time.  What bounds it: the instructions of the
// (edge, type pair) steps, each two products of typed degrees added to sums in
// LDS; HBM sees only the CSR and the output vectors.  50,000 graphs of 10 to
// 500 nodes took 116 ms in the general pipeline
// (relabelling, 4-cycle counts per edge, a wave per edge with its derivation:
// 69 ms of it) and take 4.3 ms here; 1,000 graphs 5.3 and 0.5 ms.
template <int NT, typename HT, int CLS>
__global__ void __launch_bounds__(NT)
k_small_globals(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
                const uint8_t *__restrict__ types, const int64_t *__restrict__ node_ptr,
                const int32_t *__restrict__ gL, const int64_t *__restrict__ goff,
                const uint32_t *__restrict__ list, int step, uint64_t *__restrict__ counters,
                int c_count, int c_next, int max_nodes, int L_max, uint64_t *__restrict__ out, uint32_t *__restrict__ status) {
    extern __shared__ __align__(16) unsigned char sm_small[];
    if (input_failed(status)) return;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid / WAVE;
    const SmallLds y = small_lds(max_nodes, L_max, NT);
    const int pmax = small_pairs(L_max), c3max = small_c3(L_max), c4max = small_c4(L_max);
    HT *hist = reinterpret_cast<HT *>(sm_small + y.hist);
    uint32_t *scan = reinterpret_cast<uint32_t *>(sm_small + y.scan) + wv * WAVE;
    uint64_t *masks = reinterpret_cast<uint64_t *>(sm_small + y.masks);
    uint16_t *r4tab = reinterpret_cast<uint16_t *>(sm_small + y.rank4);
    uint16_t *r3tab = reinterpret_cast<uint16_t *>(sm_small + y.rank3);
    uint16_t *pairs = reinterpret_cast<uint16_t *>(sm_small + y.pairs);
    uint16_t *triples = reinterpret_cast<uint16_t *>(sm_small + y.triples);
    uint16_t *cnt = reinterpret_cast<uint16_t *>(sm_small + y.cnt) + (size_t)wv * WAVE * L_max;
    uint32_t *equeue = reinterpret_cast<uint32_t *>(sm_small + y.pair) + 4 * wv * WAVE;
    uint32_t *cqueue = equeue + 2 * WAVE;
    uint16_t *rank = reinterpret_cast<uint16_t *>(sm_small + y.rank);
    uint32_t *row = reinterpret_cast<uint32_t *>(sm_small + y.row);
    uint8_t *ty = sm_small + y.types;
    // co-lexicographic rank tables of type multisets (the same for every
    // number of types): unordered pairs and triples in rank order, the rank
    // of two pairs together and of a pair and a type
    for (int b = tid; b < L_max; b += NT)
        for (int a = 0; a <= b; ++a) pairs[a + b * (b + 1) / 2] = (uint16_t)(a | (b << 8));
    for (int q = tid; q < L_max * L_max * L_max; q += NT) {
        const int a = q % L_max, b = (q / L_max) % L_max, c = q / (L_max * L_max);
        if (a <= b && b <= c) triples[rank3(a, b, c)] = (uint16_t)(a | (b << 4) | (c << 8));
    }
    __syncthreads();
    for (int q = tid; q < pmax * pmax; q += NT) {
        const int p = pairs[q / pmax], r = pairs[q % pmax];
        r4tab[q] = (uint16_t)rank4(p & 255, p >> 8, r & 255, r >> 8);
    }
    for (int q = tid; q < pmax * L_max; q += NT) {
        const int p = pairs[q / L_max];
        r3tab[q] = (uint16_t)rank3(p & 255, p >> 8, q % L_max);
    }
    __shared__ uint64_t s_next;
    const uint64_t count = counters[c_count];
    // graphs per queue step: enough steps to balance, few atomics on one word
    uint64_t chunk = count / ((uint64_t)gridDim.x * 8);
    chunk = chunk < 1 ? 1 : chunk > 8 ? 8 : chunk;
    uint64_t at = 0, end = 0;
    uint32_t bad = 0;
    while (true) {
        __syncthreads();   // the previous graph's output has been read
        if (at == end) {
            if (tid == 0) s_next = atomicAdd((unsigned long long *)&counters[c_next], chunk);
            __syncthreads();
            at = s_next;
            if (at >= count) break;
            end = at + chunk < count ? at + chunk : count;
        }
        const int64_t g = list[(int64_t)step * (int64_t)at];
        ++at;
        const int64_t a0 = node_ptr[g];
        const int n = (int)(node_ptr[g + 1] - a0);
        SmallGraph<HT> S;
        S.n = n;
        const int W = small_words(n);
        S.stride = small_stride(n);
        S.L = gL[g];
        S.P = small_pairs(S.L);
        S.bits = reinterpret_cast<unsigned long long *>(sm_small + y.bits);
        S.masks = masks;
        S.rank4 = r4tab;
        S.rank3 = r3tab;
        S.pairs = pairs;
        S.deg = reinterpret_cast<uint16_t *>(sm_small + y.deg);
        S.types = ty;
        S.pmax = pmax;
        S.lmax = L_max;
        S.h0 = hist;
        S.p3 = S.h0 + pmax;
        S.k3 = S.p3 + c3max;
        S.k4 = S.k3 + c3max;
        S.dia = S.k4 + c4max;
        S.tail = S.dia + c4max;
        S.c4 = S.tail + c4max;
        S.star = S.c4 + c4max;
        S.p4 = S.star + c4max;
        const int L = S.L, P = S.P, c3 = small_c3(L), c4 = small_c4(L);
        for (int q = tid; q < pmax + 2 * c3max + 6 * c4max; q += NT) hist[q] = 0;
        for (int q = tid; q < n * S.stride; q += NT) S.bits[q] = 0ull;
        for (int q = tid; q < L * W; q += NT) masks[q] = 0ull;
        const int64_t s0 = rp[a0];
        for (int v = tid; v <= n; v += NT) row[v] = (uint32_t)(rp[a0 + v] - s0);
        // ranks by degree: a counting sort (degrees are below n; the order of
        // equal degrees does not change a count)
        uint32_t *bins = equeue - 4 * wv * WAVE;   // 4 NT words
        for (int q = tid; q < n; q += NT) bins[q] = 0u;
        __syncthreads();
        for (int v = tid; v < n; v += NT) atomicAdd(&bins[row[v + 1] - row[v]], 1u);
        __syncthreads();
        if (wv == 0) {
            uint32_t carry = 0;
            for (int q0 = 0; q0 < n; q0 += WAVE) {
                const uint32_t c = q0 + lane < n ? bins[q0 + lane] : 0u;
                const uint32_t incl = wave_incl_scan(c);
                if (q0 + lane < n) bins[q0 + lane] = carry + incl - c;
                carry += __shfl(incl, WAVE - 1, WAVE);
            }
        }
        __syncthreads();
        for (int v = tid; v < n; v += NT) {
            const int r = (int)atomicAdd(&bins[row[v + 1] - row[v]], 1u);
            const int t = types[a0 + v];
            rank[v] = (uint16_t)r;
            ty[r] = (uint8_t)t;
            atomicOr(reinterpret_cast<unsigned long long *>(&masks[t * W + (r >> 6)]),
                     1ull << (r & 63));
        }
        __syncthreads();
        const uint32_t slots = n > 0 ? row[n] : 0u;
        for (uint32_t s = tid; s < slots; s += NT) {
            const int u = rank[small_row(row, n, s)];
            const int x = rank[(int)(col[s0 + s] - a0)];
            atomicOr(&S.bits[u * S.stride + (x >> 6)], 1ull << (x & 63));
        }
        __syncthreads();
        for (int q = tid; q < n * L; q += NT) {
            const int v = q / L, t = q - v * L;
            int c = 0;
            for (int z = 0; z < W; ++z) c += __popcll(S.bits[v * S.stride + z] & masks[t * W + z]);
            S.deg[q] = (uint16_t)c;
        }
        __syncthreads();
        // node terms: 3-paths and stars around each centre; each thread keeps
        // its types and walks nodes
        for (int p0 = 0; p0 < P; p0 += NT) {
            const int per = P <= NT ? NT / P : 1;
            const int sub = P <= NT ? tid / P : 0;
            const int p = P <= NT ? tid - sub * P : p0 + tid;
            if (sub >= per || p >= P) continue;
            const int t = pairs[p] & 255, u = pairs[p] >> 8;
            for (int v = sub; v < n; v += per) {
                const uint32_t dt = S.deg[v * L + t], du = S.deg[v * L + u];
                small_add(&S.p3[r3tab[p * L_max + ty[v]]], (HT)(t == u ? dt * (dt - 1) / 2 : dt * du));
            }
        }
        for (int r0 = 0; r0 < c3; r0 += NT) {
            const int per = c3 <= NT ? NT / c3 : 1;
            const int sub = c3 <= NT ? tid / c3 : 0;
            const int r = c3 <= NT ? tid - sub * c3 : r0 + tid;
            if (sub >= per || r >= c3) continue;
            const int t = triples[r] & 15, u = (triples[r] >> 4) & 15, w = triples[r] >> 8;
            const uint16_t *r4 = r4tab + small_rank2(t, u) * pmax;
            for (int v = sub; v < n; v += per) {
                const uint32_t dt = S.deg[v * L + t], du = S.deg[v * L + u], dw = S.deg[v * L + w];
                if (!dt || !du || !dw) continue;
                uint32_t x;   // below 512^3
                if (t == u && u == w) x = dt * (dt - 1) * (dt - 2) / 6;
                else if (t == u) x = dt * (dt - 1) / 2 * dw;
                else if (u == w) x = dt * (du * (du - 1) / 2);
                else x = dt * du * dw;
                small_add(&S.star[r4[small_rank2(w, ty[v])]], (HT)x);
            }
        }
        switch (W) {
            case 1:
                if constexpr (CLS == 0)
                    small_all_pairs<1, NT>(S, equeue, cqueue, cnt, scan);
                break;
            case 2:
                if constexpr (CLS == 0)
                    small_all_pairs<2, NT>(S, equeue, cqueue, cnt, scan);
                break;
            case 4:
                if constexpr (CLS == 1)
                    small_all_pairs<4, NT>(S, equeue, cqueue, cnt, scan);
                break;
            default:
                if constexpr (CLS == 2)
                    small_all_pairs<8, NT>(S, equeue, cqueue, cnt, scan);
        }
        __syncthreads();
        // induced counts per multiset, in the graph's own layout
        uint64_t *dst = out + goff[g];
        for (int q = tid; q < P; q += NT) dst[q] = S.h0[q];
        for (int q = tid; q < c3; q += NT) {
            const uint64_t k3 = S.k3[q];
            if (k3 % 3) bad |= ST_NOT_DIVISIBLE;
            const int64_t h1 = (int64_t)S.p3[q] - (int64_t)k3;   // three copies per triangle
            if (h1 < 0) bad |= ST_INTERNAL;
            dst[P + q] = (uint64_t)h1;
            dst[P + c3 + q] = k3 / 3;
        }
        for (int q = tid; q < c4; q += NT) {
            if (S.tail[q] & 1) bad |= ST_NOT_DIVISIBLE;
            const int64_t h8 = (int64_t)S.k4[q];
            const int64_t h7 = (int64_t)S.dia[q] - 6 * h8;
            const int64_t h6 = (int64_t)(S.tail[q] / 2) - 4 * h7 - 12 * h8;
            const int64_t h5 = (int64_t)S.c4[q] - h7 - 3 * h8;
            const int64_t h4 = (int64_t)S.star[q] - h6 - 2 * h7 - 4 * h8;
            const int64_t h3 = (int64_t)S.p4[q] - 4 * h5 - 2 * h6 - 6 * h7 - 12 * h8;
            if (h7 < 0 || h6 < 0 || h5 < 0 || h4 < 0 || h3 < 0) bad |= ST_INTERNAL;
            const int64_t h[6] = {h3, h4, h5, h6, h7, h8};
#pragma unroll
            for (int z = 0; z < 6; ++z) dst[P + 2 * c3 + z * c4 + q] = (uint64_t)h[z];
        }
    }
    bad = wave_or(bad);
    if (lane == 0 && bad) atomicOr(status, bad);
}

// The path is taken when the largest graph fits a CU's LDS beside the static
// words (512 nodes with up to 10 types, fewer nodes with more types).
bool small_batch_fits(int64_t max_nodes, int L_max) {
    if (max_nodes > SMALL_NODES) return false;
    const int64_t mid = max_nodes < SMALL_MID ? max_nodes : SMALL_MID;
    const int64_t lo = max_nodes < SMALL_LO ? max_nodes : SMALL_LO;
    return small_lds((int)max_nodes, L_max, SMALL_NT_HI).total <= 156 * 1024 &&
           small_lds((int)mid, L_max, 2 * SMALL_NT_MID).total <= 156 * 1024 &&
           small_lds((int)lo, L_max, 2 * SMALL_NT_LO).total <= 156 * 1024;
}

namespace {
struct SmallLaunch {
    const int64_t *rp;
    const int32_t *col;
    const uint8_t *types;
    int64_t n, nnz;
    const BatchIn *b;
    uint64_t *counters;
    int L_max, cus;
    uint64_t *out;
    uint32_t *status;
    hipStream_t st;
};

hipError_t small_check(const SmallLaunch &a, const uint32_t *list, int step, int c_count,
                       int max_nodes) {
    const size_t lds = sizeof(uint64_t) * (size_t)max_nodes * small_stride(max_nodes) +
                       sizeof(uint32_t) * (size_t)(max_nodes + 1);
    int64_t grid = (int64_t)a.cus * 8;
    if (grid > a.b->G) grid = a.b->G;
    k_small_check<<<(unsigned)grid, SMALL_THREADS, lds, a.st>>>(
        a.rp, a.col, a.types, a.b->node_ptr, a.b->gL, list, step, a.counters, c_count, max_nodes,
        a.n, a.nnz, a.status);
    return hipGetLastError();
}

template <int NT, typename HT, int CLS>
hipError_t small_globals(const SmallLaunch &a, const uint32_t *list, int step, int c_count,
                         int c_next, int max_nodes) {
    const size_t lds = small_lds(max_nodes, a.L_max, NT).total;
    // workgroups that fit the chip at once pull graphs from a queue
    int64_t per_cu = (int64_t)(160 * 1024) / (int64_t)(lds + 64);
    if (per_cu > 2048 / NT) per_cu = 2048 / NT;
    if (per_cu < 1) per_cu = 1;
    int64_t grid = (int64_t)a.cus * per_cu;
    if (grid > a.b->G) grid = a.b->G;
    k_small_globals<NT, HT, CLS><<<(unsigned)grid, NT, lds, a.st>>>(
        a.rp, a.col, a.types, a.b->node_ptr, a.b->gL, a.b->goff, list, step, a.counters, c_count,
        c_next, max_nodes, a.L_max, a.out, a.status);
    return hipGetLastError();
}
}  // namespace

// list and counters: k_batch_graphs's lists by size (C_A_LIGHT, C_B_LIGHT and
// C_A_HEAVY graphs).  Every graph is checked before the first output is written.
hipError_t launch_small_batch(const int64_t *rp, const int32_t *col, const uint8_t *types,
                              int64_t n, int64_t nnz, const BatchIn &b, int max_nodes, int L_max,
                              int cus, const uint32_t *list, uint64_t *counters, uint64_t *out,
                              uint32_t *status, hipStream_t st) {
    const SmallLaunch a{rp, col, types, n, nnz, &b, counters, L_max, cus, out, status, st};
    const uint32_t *lists[3] = {list, list + b.G, list + 2 * b.G - 1};
    const int steps[3] = {1, 1, -1}, counts[3] = {C_A_LIGHT, C_B_LIGHT, C_A_HEAVY};
    const int bounds[3] = {SMALL_LO, SMALL_MID, SMALL_NODES};
    const bool few = b.G <= (int64_t)SMALL_FEW * cus;
    for (int pass = 0; pass < 2; ++pass)
        for (int q = 2; q >= 0; --q) {
            if (q > 0 && max_nodes <= bounds[q - 1]) continue;
            const int most = max_nodes < bounds[q] ? max_nodes : bounds[q];
            hipError_t e;
            if (pass == 0) e = small_check(a, lists[q], steps[q], counts[q], most);
            else if (q == 2)
                e = small_globals<SMALL_NT_HI, unsigned long long, 2>(a, lists[q], steps[q], counts[q],
                                                                   C_A_NEXT, most);
            else if (q == 1 && few)
                e = small_globals<2 * SMALL_NT_MID, uint32_t, 1>(a, lists[q], steps[q], counts[q],
                                                                 C_B_NEXT, most);
            else if (q == 1)
                e = small_globals<SMALL_NT_MID, uint32_t, 1>(a, lists[q], steps[q], counts[q],
                                                             C_B_NEXT, most);
            else if (few)
                e = small_globals<2 * SMALL_NT_LO, uint32_t, 0>(a, lists[q], steps[q], counts[q],
                                                                C_EDGE_NEXT, most);
            else
                e = small_globals<SMALL_NT_LO, uint32_t, 0>(a, lists[q], steps[q], counts[q],
                                                            C_EDGE_NEXT, most);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

}  // namespace tg
