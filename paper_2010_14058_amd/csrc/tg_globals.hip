// Global typed counts of a single graph without its per-edge table.
//
// The global vector follows, per type multiset, from sums of not necessarily
// induced copies (the relations in tg_small.hip), so that none of the per-edge
// quantities behind the rows is needed beyond the typed triangle counts:
//   P3, STAR   node sums of products of typed degrees;
//   P4, TAIL   node sums of products of typed degrees with the node aggregates
//              D and A (each path met from both its middle nodes, each tailed
//              triangle over both edges at its corner: halved at the end);
//   K3, DIA    edge sums of typed triangle counts and of their products;
//   C4         the wedge counts of pass A: every 4-cycle once, at its top node,
//              counted over ordered centre pairs (halved at the end); pass B and
//              the per-edge credits fall away;
//   K4         the adjacent pairs above an edge's larger end in its triangle
//              set: every clique once, at its two lowest nodes, where the
//              per-edge counts meet it six times with the whole set.
#include <hip/hip_runtime.h>

#include "tg_device.hpp"

namespace tg {

constexpr int GLOB_THREADS = 256;
constexpr int GLOB_L = GLOBALS_MAX_L;
constexpr int PAIR_LIST = 32;   // hub members tested pair by pair up to this many
constexpr int LOW_LIST = 256;   // low members listed in LDS, more are taken one by one

__device__ __forceinline__ int grank2(int a, int b) {
    return a <= b ? a + b * (b + 1) / 2 : b + a * (a + 1) / 2;
}

// Rank of every two unordered type pairs together, by the pairs' own ranks.
__global__ void k_rank4_table(int L, uint16_t *__restrict__ r4) {
    const int P = L * (L + 1) / 2;
    for (int q = threadIdx.x; q < P * P; q += blockDim.x) {
        int p[2] = {q / P, q % P}, lo[2], hi[2];
        for (int z = 0; z < 2; ++z) {
            int h = 0;
            while ((h + 1) * (h + 2) / 2 <= p[z]) ++h;
            hi[z] = h;
            lo[z] = p[z] - h * (h + 1) / 2;
        }
        r4[q] = (uint16_t)rank4(lo[0], hi[0], lo[1], hi[1]);
    }
}

// Sections of one copy of the sums.
struct GlobSections {
    int n2, n3, n4;
    __host__ __device__ explicit GlobSections(int L)
        : n2(L * (L + 1) / 2), n3(L * (L + 1) * (L + 2) / 6),
          n4(L * (L + 1) / 2 * (L + 2) / 3 * (L + 3) / 4) {}
    __host__ __device__ int h0() const { return 0; }
    __host__ __device__ int p3() const { return n2; }
    __host__ __device__ int k3() const { return n2 + n3; }
    __host__ __device__ int k4() const { return n2 + 2 * n3; }
    __host__ __device__ int dia() const { return k4() + n4; }
    __host__ __device__ int tail() const { return k4() + 2 * n4; }
    __host__ __device__ int c4() const { return k4() + 3 * n4; }
    __host__ __device__ int star() const { return k4() + 4 * n4; }
    __host__ __device__ int p4() const { return k4() + 5 * n4; }
    __host__ __device__ int words() const { return k4() + 6 * n4; }
};

int globals_words(int L) { return GlobSections(L).words(); }
int globals_c4(int L) { return GlobSections(L).c4(); }

__device__ __forceinline__ void gsum(unsigned long long *p, uint64_t v) {
    if (v) atomicAdd(p, (unsigned long long)v);
}

// Node sums.  A thread keeps its types (t, u) or (b, u, t) and walks the
// workgroup's nodes; sums meet in LDS.
__global__ void __launch_bounds__(GLOB_THREADS)
k_node_globals(const uint8_t *__restrict__ ntype, const uint32_t *__restrict__ tdeg,
               const uint32_t *__restrict__ A, const uint32_t *__restrict__ D, int64_t n, int L,
               const uint16_t *__restrict__ r4g, uint64_t *__restrict__ acc, int copies,
               const uint32_t *__restrict__ status) {
    extern __shared__ unsigned long long sm_glob[];
    if (input_failed(status)) return;
    const GlobSections S(L);
    const int tid = threadIdx.x, LL = L * L, P = S.n2, LP = tri_pitch(L);
    unsigned long long *sum = sm_glob;
    uint16_t *r4 = reinterpret_cast<uint16_t *>(sum + S.words());
    for (int q = tid; q < S.words(); q += GLOB_THREADS) sum[q] = 0ull;
    for (int q = tid; q < P * P; q += GLOB_THREADS) r4[q] = r4g[q];
    __syncthreads();
    unsigned long long *p3 = sum + S.p3(), *star = sum + S.star(), *p4 = sum + S.p4(),
                       *tail = sum + S.tail();
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    const int64_t v0 = (int64_t)blockIdx.x * per, v1 = v0 + per < n ? v0 + per : n;
    // P3: pairs of neighbours
    {
        const int groups = GLOB_THREADS / P, g = tid / P, p = tid - g * P;
        if (g < groups) {
            int u = 0;
            while ((u + 1) * (u + 2) / 2 <= p) ++u;
            const int t = p - u * (u + 1) / 2;
            for (int64_t v = v0 + g; v < v1; v += groups) {
                const uint64_t dt = tdeg[v * LP + t], du = tdeg[v * LP + u];
                if (!dt || !du) continue;
                gsum(&p3[rank3(t, u, ntype[v])], t == u ? dt * (dt - 1) / 2 : dt * du);
            }
        }
    }
    // STAR: triples of neighbours
    for (int r0 = 0; r0 < S.n3; r0 += GLOB_THREADS) {
        const int groups = S.n3 <= GLOB_THREADS ? GLOB_THREADS / S.n3 : 1;
        const int g = S.n3 <= GLOB_THREADS ? tid / S.n3 : 0;
        const int r = S.n3 <= GLOB_THREADS ? tid - g * S.n3 : r0 + tid;
        if (g >= groups || r >= S.n3) continue;
        int w = 0;
        while ((w + 1) * (w + 2) * (w + 3) / 6 <= r) ++w;
        const int p = r - w * (w + 1) * (w + 2) / 6;
        int u = 0;
        while ((u + 1) * (u + 2) / 2 <= p) ++u;
        const int t = p - u * (u + 1) / 2;
        for (int64_t v = v0 + g; v < v1; v += groups) {
            const uint64_t dt = tdeg[v * LP + t], du = tdeg[v * LP + u], dw = tdeg[v * LP + w];
            if (!dt || !du || !dw) continue;
            uint64_t x;   // degrees below 2^16
            if (t == w) x = dt * (dt - 1) / 2 * (dt - 2) / 3;
            else if (t == u) x = dt * (dt - 1) / 2 * dw;
            else if (u == w) x = dt * (du * (du - 1) / 2);
            else x = dt * du * dw;
            gsum(&star[r4[grank2(t, u) * P + grank2(w, ntype[v])]], x);
        }
    }
    // P4 and TAIL: neighbour k of type b with a second node of type u (its
    // neighbour, or a common one), and another neighbour of type t of v
    for (int r0 = 0; r0 < LL * L; r0 += GLOB_THREADS) {
        const int groups = LL * L <= GLOB_THREADS ? GLOB_THREADS / (LL * L) : 1;
        const int g = LL * L <= GLOB_THREADS ? tid / (LL * L) : 0;
        const int r = LL * L <= GLOB_THREADS ? tid - g * LL * L : r0 + tid;
        if (g >= groups || r >= LL * L) continue;
        const int t = r / LL, b = (r - t * LL) / L, u = r % L;
        const int tu = grank2(t, u);
        for (int64_t v = v0 + g; v < v1; v += groups) {
            const int a = ntype[v];
            const int64_t db = tdeg[v * LP + b];
            if (!db) continue;
            const int64_t dt = tdeg[v * LP + t];
            const int64_t Ab = A[v * LL + b * L + u], Db = D[v * LL + b * L + u];
            const int at = r4[grank2(a, b) * P + tu];
            // k's neighbours of type u without v, times v's of type t without
            // k; of these pairs the one common node is no path (t == u)
            const int64_t paths = (Db - (u == a ? db : 0)) * (dt - (t == b)) - (t == u ? Ab : 0);
            const int64_t tails = Ab * (dt - (t == b) - (t == u));
            gsum(&p4[at], (uint64_t)paths);
            gsum(&tail[at], (uint64_t)tails);
        }
    }
    __syncthreads();
    uint64_t *out = acc + (size_t)(blockIdx.x % (unsigned)copies) * S.words();
    for (int q = tid; q < S.words(); q += GLOB_THREADS)
        if (sum[q]) atomicAdd((unsigned long long *)&out[q], sum[q]);
}

// Edge sums: the edges by type pair, typed triangles, pairs of triangles.
__global__ void __launch_bounds__(GLOB_THREADS)
k_edge_globals(const uint8_t *__restrict__ ntype, const int32_t *__restrict__ ei,
               const int32_t *__restrict__ ej, const uint32_t *__restrict__ tri,
               const uint32_t *__restrict__ ttot, int64_t m, int L,
               const uint16_t *__restrict__ r4g, uint64_t *__restrict__ acc, int copies,
               const uint32_t *__restrict__ status) {
    extern __shared__ unsigned long long sm_glob[];
    __shared__ uint32_t todo[GLOB_THREADS], todo_ab[GLOB_THREADS];
    __shared__ int have;
    if (input_failed(status)) return;
    const GlobSections S(L);
    const int tid = threadIdx.x, P = S.n2;
    unsigned long long *sum = sm_glob;   // h0, then k3 and dia
    unsigned long long *k3 = sum + S.n2, *dia = k3 + S.n3;
    uint16_t *r4 = reinterpret_cast<uint16_t *>(dia + S.n4);
    for (int q = tid; q < S.n2 + S.n3 + S.n4; q += GLOB_THREADS) sum[q] = 0ull;
    for (int q = tid; q < P * P; q += GLOB_THREADS) r4[q] = r4g[q];
    const int groups = GLOB_THREADS / P, g = tid / P, p = tid - g * P;
    int u = 0;
    while ((u + 1) * (u + 2) / 2 <= p) ++u;
    const int t = p - u * (u + 1) / 2;
    for (int64_t e0 = (int64_t)blockIdx.x * GLOB_THREADS; e0 < m;
         e0 += (int64_t)gridDim.x * GLOB_THREADS) {
        if (tid == 0) have = 0;
        __syncthreads();
        const int64_t e = e0 + tid;
        if (e < m) {
            const int ab = grank2(ntype[ei[e]], ntype[ej[e]]);
            atomicAdd(&sum[ab], 1ull);
            if (ttot[e]) {
                const int at = atomicAdd(&have, 1);
                todo[at] = (uint32_t)tid;
                todo_ab[at] = (uint32_t)ab;
            }
        }
        __syncthreads();
        // the edges with triangles, one (edge, type pair) per thread
        if (g < groups)
            for (int q = g; q < have; q += groups) {
                const uint32_t *T = tri + (size_t)(e0 + todo[q]) * L;
                const uint64_t ct = T[t], cu = T[u];
                const int ab = (int)todo_ab[q];
                gsum(&dia[r4[ab * P + p]], t == u ? ct * (ct - (ct ? 1 : 0)) / 2 : ct * cu);
                if (t == u && ct) {
                    int hi = 0;
                    while ((hi + 1) * (hi + 2) / 2 <= ab) ++hi;
                    atomicAdd(&k3[rank3(ab - hi * (hi + 1) / 2, hi, t)], (unsigned long long)ct);
                }
            }
        __syncthreads();
    }
    uint64_t *out = acc + (size_t)(blockIdx.x % (unsigned)copies) * S.words();
    for (int q = tid; q < S.n2 + S.n3 + S.n4; q += GLOB_THREADS) {
        if (!sum[q]) continue;
        const int at = q < S.n2 ? S.h0() + q : q < S.n2 + S.n3 ? S.k3() + (q - S.n2)
                                                               : S.dia() + (q - S.n2 - S.n3);
        atomicAdd((unsigned long long *)&out[at], sum[q]);
    }
}

// 4-cliques, one wave per listed edge (i < j by rank): the members of its
// triangle set above j -- hubs as bits, two words per lane; low nodes listed in
// order of rank -- and their adjacent pairs: the rows of the low members above
// themselves, 64 of them laid end to end, each entry looked up in the bits or
// the list.  One member's row after the other, looked up in the rows of both
// ends, kept most lanes idle and took 65 ms for 4M edges in cliques of 64
// nodes, where the per-edge counts take 47; 18 ms now.
__global__ void __launch_bounds__(WAVE)
k_cliques4(EdgeArgs a, const uint32_t *__restrict__ eslot, const uint16_t *__restrict__ r4g,
           uint64_t *__restrict__ acc, int copies) {
    extern __shared__ unsigned long long sm_glob[];
    __shared__ unsigned long long Tm[HUB_MAX / 64];
    __shared__ uint16_t list[PAIR_LIST];
    __shared__ int32_t low[LOW_LIST];
    __shared__ uint8_t low_type[LOW_LIST];
    __shared__ uint32_t scan[WAVE];
    __shared__ int64_t first[WAVE];
    if (input_failed(a.status)) return;
    const uint64_t count = a.counters[C_EDGE_FEW];
    if (blockIdx.x >= count) return;
    const int L = a.L, lane = threadIdx.x, Hw = a.Hw, TP = tm_pitch(L);
    const GlobSections S(L);
    const int P = S.n2;
    unsigned long long *sum = sm_glob;
    uint16_t *r4 = reinterpret_cast<uint16_t *>(sum + S.n4);
    for (int q = lane; q < S.n4; q += WAVE) sum[q] = 0ull;
    for (int q = lane; q < P * P; q += WAVE) r4[q] = r4g[q];
    // this lane's words of the hub type masks
    unsigned long long tm[2][GLOB_L];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        const int w = lane + z * WAVE;
        unsigned long long rest = ~0ull;
#pragma unroll
        for (int t = 0; t < GLOB_L; ++t) {
            tm[z][t] = 0ull;
            if (t < L - 1 && w < Hw) tm[z][t] = a.TM[(size_t)w * TP + t];
            rest &= ~tm[z][t];
        }
#pragma unroll
        for (int t = 0; t < GLOB_L; ++t)
            if (t == L - 1) tm[z][t] = rest;
    }
    const int32_t base = a.hub_base;
    wave_sync();
    for (uint64_t q = blockIdx.x; q < count; q += gridDim.x) {
        const int64_t e = a.few_list[q];
        const int32_t i = a.ei[e], j = a.ej[e];
        const int32_t lo = i < j ? i : j, hi = i < j ? j : i;
        // the rows above hi
        const int64_t lb = (int64_t)eslot[2 * (size_t)e] + 1, le = a.nrp[lo + 1];
        const int64_t hb = a.nrp[hi] + a.nlow[hi], he = a.nrp[hi + 1];
        if (le - lb < 2 || he - hb < 2) continue;
        const uint16_t *rt = r4 + grank2(a.ntype[lo], a.ntype[hi]) * P;
        const int64_t lh = a.hstart[lo] > lb ? a.hstart[lo] : lb;
        const int64_t hh = a.hstart[hi] > hb ? a.hstart[hi] : hb;
        // hub members
        unsigned long long T[2] = {0ull, 0ull};
        if (lo >= base) {
            const uint64_t *rl = a.HB + (size_t)(lo - base) * Hw, *rh = a.HB + (size_t)(hi - base) * Hw;
            const int hx = hi - base;
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                const int w = lane + z * WAVE;
                if (w >= Hw || w < (hx >> 6)) continue;
                T[z] = rl[w] & rh[w];
                if (w == (hx >> 6)) T[z] &= (hx & 63) == 63 ? 0ull : ~0ull << ((hx & 63) + 1);
            }
        } else if (lh < le && hh < he) {
            for (int w = lane; w < Hw; w += WAVE) Tm[w] = 0ull;
            wave_sync();
            const bool lo_walks = le - lh <= he - hh;
            const int64_t wb = lo_walks ? lh : hh, we = lo_walks ? le : he;
            const int64_t ob = lo_walks ? hh : lh, oe = lo_walks ? he : le;
            const int32_t other = lo_walks ? hi : lo;
            for (int64_t p = wb + lane; p < we; p += WAVE) {
                const int32_t x = a.ncol[p];
                const int hx = x - base;
                bool found;
                if (other >= base) {
                    found = (a.HB[(size_t)(other - base) * Hw + (hx >> 6)] >> (hx & 63)) & 1ull;
                } else {
                    const int64_t at = lower_bound(a.ncol, ob, oe, x);
                    found = at < oe && a.ncol[at] == x;
                }
                if (found) atomicOr(&Tm[hx >> 6], 1ull << (hx & 63));
            }
            wave_sync();
#pragma unroll
            for (int z = 0; z < 2; ++z)
                if (lane + z * WAVE < Hw) T[z] = Tm[lane + z * WAVE];
        }
        const uint32_t mine = (uint32_t)(__popcll(T[0]) + __popcll(T[1]));
        const uint32_t incl = wave_incl_scan(mine);
        const uint32_t nh = __shfl(incl, WAVE - 1, WAVE);
        if (nh >= 2 && nh <= (uint32_t)PAIR_LIST) {
            uint32_t at = incl - mine;
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                unsigned long long m = T[z];
                while (m) {
                    const int b = __ffsll((long long)m) - 1;
                    m &= m - 1;
                    list[at++] = (uint16_t)((lane + z * WAVE) * 64 + b);
                }
            }
            wave_sync();
            const int pairs = (int)(nh * (nh - 1) / 2);
            for (int f = lane; f < pairs; f += WAVE) {
                int y = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)f)) * 0.5f);
                while (y * (y - 1) / 2 > f) --y;
                while ((y + 1) * y / 2 <= f) ++y;
                const int hx = list[f - y * (y - 1) / 2], hy = list[y];
                if ((a.HB[(size_t)hx * Hw + (hy >> 6)] >> (hy & 63)) & 1ull)
                    atomicAdd(&sum[rt[grank2(a.ntype[base + hx], a.ntype[base + hy])]], 1ull);
            }
            wave_sync();
        } else if (nh > (uint32_t)PAIR_LIST) {
            // members of one type at a time, each one's bit row against the
            // set's bits above it
            for (int tx = 0; tx < L; ++tx) {
                uint32_t cnt[GLOB_L];
#pragma unroll
                for (int t = 0; t < GLOB_L; ++t) cnt[t] = 0u;
                bool any = false;
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    unsigned long long x = 0ull;
#pragma unroll
                    for (int t = 0; t < GLOB_L; ++t)
                        if (t == tx) x = T[z] & tm[z][t];
                    uint64_t words = __ballot(x != 0ull);
                    any |= words != 0ull;
                    while (words) {
                        const int src = __ffsll((long long)words) - 1;
                        words &= words - 1;
                        unsigned long long m = __shfl(x, src, WAVE);
                        while (m) {
                            const int b = __ffsll((long long)m) - 1;
                            m &= m - 1;
                            const int w = src + z * WAVE;       // the member is hub 64 w + b
                            const uint64_t *row = a.HB + (size_t)(w * 64 + b) * Hw;
#pragma unroll
                            for (int y = 0; y < 2; ++y) {
                                const int v = lane + y * WAVE;
                                unsigned long long r = v < Hw && v >= w ? row[v] & T[y] : 0ull;
                                if (v == w) r &= b == 63 ? 0ull : ~0ull << (b + 1);
#pragma unroll
                                for (int t = 0; t < GLOB_L; ++t)
                                    if (t < L) cnt[t] += (uint32_t)__popcll(r & tm[y][t]);
                            }
                        }
                    }
                }
                if (!any) continue;
#pragma unroll
                for (int t = 0; t < GLOB_L; ++t) {
                    if (t >= L) break;
                    uint32_t c = cnt[t];
#pragma unroll
                    for (int d = WAVE / 2; d > 0; d >>= 1) c += __shfl_xor(c, d, WAVE);
                    if (lane == 0 && c) atomicAdd(&sum[rt[grank2(tx, t)]], (unsigned long long)c);
                }
            }
        }
        if (hi >= base) continue;
        // low members x (above hi, below the hub core) and the members y > x
        const int64_t ll = a.hstart[lo], hl = a.hstart[hi];
        if (ll <= lb || hl <= hb) continue;
        if (lh < le && hh < he) {
            // the hub members' bits stand in Tm
        } else {
            for (int w = lane; w < Hw; w += WAVE) Tm[w] = 0ull;
            wave_sync();
        }
        const bool lo_walks = ll - lb <= hl - hb;
        const int64_t wb = lo_walks ? lb : hb, we = lo_walks ? ll : hl;
        const int64_t ob = lo_walks ? hb : lb, oe = lo_walks ? hl : ll;
        auto member = [&](int64_t p, int32_t &x) {
            if (p >= we) return false;
            x = a.ncol[p];
            const int64_t at = lower_bound(a.ncol, ob, oe, x);
            return at < oe && a.ncol[at] == x;
        };
        int nl = 0;
        for (int64_t p0 = wb; p0 < we && nl <= LOW_LIST; p0 += WAVE) {
            int32_t x = 0;
            const bool found = member(p0 + lane, x);
            const uint64_t bal = __ballot(found);
            const int at = nl + __popcll(bal & ((1ull << lane) - 1ull));
            if (found && at < LOW_LIST) {
                low[at] = x;
                low_type[at] = a.ctype[p0 + lane];
            }
            nl += __popcll(bal);
        }
        wave_sync();
        if (nl <= LOW_LIST) {
            for (int c0 = 0; c0 < nl; c0 += WAVE) {
                const int items = nl - c0 < WAVE ? nl - c0 : WAVE;
                uint32_t len = 0;
                if (lane < items) {
                    const int64_t x = low[c0 + lane], b = a.nrp[x] + a.nlow[x];
                    len = (uint32_t)(a.nrp[x + 1] - b);
                    first[lane] = b;
                }
                const uint32_t incl = wave_incl_scan(len);
                scan[lane] = incl;
                const uint32_t total = __shfl(incl, WAVE - 1, WAVE);
                wave_sync();
                int o = 0;
                for (uint32_t f = lane; f < total; f += WAVE) {
                    o = owner_next(scan, items, f, o);
                    const int64_t s = first[o] + (f - (o ? scan[o - 1] : 0u));
                    const int32_t y = a.ncol[s];
                    bool in;
                    if (y >= base) {
                        const int hy = y - base;
                        in = (Tm[hy >> 6] >> (hy & 63)) & 1ull;
                    } else {
                        int l = c0 + o + 1, h = nl;   // members above this one
                        while (l < h) {
                            const int mid = (l + h) >> 1;
                            if (low[mid] < y) l = mid + 1; else h = mid;
                        }
                        in = l < nl && low[l] == y;
                    }
                    if (in) atomicAdd(&sum[rt[grank2(low_type[c0 + o], a.ctype[s])]], 1ull);
                }
                wave_sync();
            }
            continue;
        }
        for (int64_t p0 = wb; p0 < we; p0 += WAVE) {
            int32_t x = 0;
            uint64_t bal = __ballot(member(p0 + lane, x));
            while (bal) {
                const int src = __ffsll((long long)bal) - 1;
                bal &= bal - 1;
                const int32_t xx = __shfl(x, src, WAVE);
                const int tx = a.ntype[xx];
                for (int64_t s = a.nrp[xx] + a.nlow[xx] + lane; s < a.nrp[xx + 1]; s += WAVE) {
                    const int32_t y = a.ncol[s];
                    bool in;
                    if (y >= base) {
                        const int hy = y - base;
                        in = (Tm[hy >> 6] >> (hy & 63)) & 1ull;
                    } else {
                        const int64_t p1 = lower_bound(a.ncol, lb, ll, y);
                        in = p1 < ll && a.ncol[p1] == y;
                        if (in) {
                            const int64_t p2 = lower_bound(a.ncol, hb, hl, y);
                            in = p2 < hl && a.ncol[p2] == y;
                        }
                    }
                    if (in) atomicAdd(&sum[rt[grank2(tx, a.ctype[s])]], 1ull);
                }
            }
        }
        wave_sync();
    }
    wave_sync();
    uint64_t *out = acc + (size_t)(blockIdx.x % (unsigned)copies) * S.words() + S.k4();
    for (int q = lane; q < S.n4; q += WAVE)
        if (sum[q]) atomicAdd((unsigned long long *)&out[q], sum[q]);
}

// The copies (at most 64, one per lane) added up, the doubled sums halved, and
// the induced counts; one wave per entry rank.
__global__ void __launch_bounds__(256)
k_globals_finalize(const uint64_t *__restrict__ acc, int copies, int L, uint64_t *__restrict__ out,
                   uint32_t *__restrict__ status) {
    if (input_failed(status)) return;
    const GlobSections S(L);
    const int lane = lane_id();
    const int q = blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
    const size_t W = (size_t)S.words();
    auto total = [&](int at) {
        return wave_sum_u64(lane < copies ? acc[(size_t)lane * W + at] : 0ull);
    };
    uint32_t bad = 0;
    if (q < S.n2) {
        const uint64_t h0 = total(S.h0() + q);
        if (lane == 0) out[q] = h0;
    }
    if (q < S.n3) {
        const uint64_t k3 = total(S.k3() + q), p3 = total(S.p3() + q);
        if (k3 % 3) bad |= ST_NOT_DIVISIBLE;
        if (p3 < k3) bad |= ST_INTERNAL;
        if (lane == 0) {
            out[S.n2 + q] = p3 - k3;            // three 3-path copies per triangle
            out[S.n2 + S.n3 + q] = k3 / 3;
        }
    }
    if (q < S.n4) {
        const uint64_t tail = total(S.tail() + q), c4 = total(S.c4() + q), p4 = total(S.p4() + q);
        if ((tail | c4 | p4) & 1) bad |= ST_NOT_DIVISIBLE;
        const int64_t h8 = (int64_t)total(S.k4() + q);
        const int64_t h7 = (int64_t)total(S.dia() + q) - 6 * h8;
        const int64_t h6 = (int64_t)(tail / 2) - 4 * h7 - 12 * h8;
        const int64_t h5 = (int64_t)(c4 / 2) - h7 - 3 * h8;
        const int64_t h4 = (int64_t)total(S.star() + q) - h6 - 2 * h7 - 4 * h8;
        const int64_t h3 = (int64_t)(p4 / 2) - 4 * h5 - 2 * h6 - 6 * h7 - 12 * h8;
        if (h7 < 0 || h6 < 0 || h5 < 0 || h4 < 0 || h3 < 0) bad |= ST_INTERNAL;
        const int64_t h[6] = {h3, h4, h5, h6, h7, h8};
#pragma unroll
        for (int z = 0; z < 6; ++z)
            if (lane == z) out[S.n2 + 2 * S.n3 + z * S.n4 + q] = (uint64_t)h[z];
    }
    if (lane == 0 && bad) atomicOr(status, bad);
}

hipError_t launch_rank4_table(int L, uint16_t *r4, hipStream_t st) {
    k_rank4_table<<<1, 256, 0, st>>>(L, r4);
    return hipGetLastError();
}

hipError_t launch_globals(const EdgeArgs &a, const uint32_t *eslot, const uint16_t *r4,
                          uint64_t *acc, int copies, int cus, uint64_t *out, hipStream_t st) {
    const GlobSections S(a.L);
    const int most = S.n4 > S.n3 ? S.n4 : S.n3;   // n2 <= n3 <= n4
    const size_t table = sizeof(uint16_t) * (size_t)S.n2 * S.n2;
    hipError_t e = launch_edge_classes(a, cus, st, true);
    if (e != hipSuccess) return e;
    int64_t grid = (a.n + 63) / 64;
    if (grid > 4 * (int64_t)cus) grid = 4 * (int64_t)cus;
    k_node_globals<<<(unsigned)grid, GLOB_THREADS, sizeof(uint64_t) * (size_t)S.words() + table, st>>>(
        a.ntype, a.tdeg, reinterpret_cast<const uint32_t *>(a.A),
        reinterpret_cast<const uint32_t *>(a.D), a.n, a.L, r4, acc, copies, a.status);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.m > 0) {
        grid = (a.m + GLOB_THREADS - 1) / GLOB_THREADS;
        if (grid > 4 * (int64_t)cus) grid = 4 * (int64_t)cus;
        k_edge_globals<<<(unsigned)grid, GLOB_THREADS,
                         sizeof(uint64_t) * (size_t)(S.n2 + S.n3 + S.n4) + table, st>>>(
            a.ntype, a.ei, a.ej, a.tri, a.ttot, a.m, a.L, r4, acc, copies, a.status);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        grid = a.m < 32 * (int64_t)cus ? a.m : 32 * (int64_t)cus;
        k_cliques4<<<(unsigned)grid, WAVE, sizeof(uint64_t) * (size_t)S.n4 + table, st>>>(
            a, eslot, r4, acc, copies);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_globals_finalize<<<(unsigned)((most + 3) / 4), 256, 0, st>>>(acc, copies, a.L, out,
                                                                      a.status);
    return hipGetLastError();
}

}  // namespace tg
