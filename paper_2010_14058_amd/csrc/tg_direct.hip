// Single graphs of few edges: every edge counted from its own neighbourhood,
// with no relabelling, no per-edge intermediate tables and five launches.
//
// For an edge (u, v) the other nodes fall into S_u, S_v, T (Cor. 1, 2) and the
// rest; each adjacent pair with a node k in S_u, S_v or T is seen by walking
// k's row, and its orbit follows from the classes of its two ends (Alg. 2 and
// 3 as enumerations: g3, g6, g7, g8, g10, g12); Lemmas 1-4 give the others.
// The walk costs sum over k of d_k steps per edge, D = sum over nodes u of
// d_u sum over neighbours k of d_k steps in all, more than the general
// pipeline's degree-ordered wedges, but a small graph's time is launches and
// dependent passes, not steps.
#include <hip/hip_runtime.h>

#include "tg_device.hpp"

namespace tg {

constexpr int DIRECT_WAVES = 4;
constexpr int DIRECT_THREADS = DIRECT_WAVES * WAVE;
constexpr int DIRECT_MOST = 16;   // most waves of an edge workgroup
// Copies of the global sums, so that few workgroups add to the same words.
constexpr int DIRECT_COPIES = 16;
// Copies of an edge's orbit counters: lanes of one step mostly count the same
// few type pairs.
constexpr int ORBIT_COPIES = 4;
// 32-bit orbit counters (at most one per walk step), 16-bit ids of near nodes.
static_assert(DIRECT_STEPS <= 0xffffffffu && DIRECT_NODES <= 65536, "counter and id widths");

// Checks of one input row per wave: order, range, self-loops, types, and each
// neighbour's row holding the mirrored entry; entries above the diagonal;
// the walk's steps and the largest degree (C_DIRECT_STEPS, C_DIRECT_DEG).
// Also clears the copies of the global sums.
__global__ void __launch_bounds__(DIRECT_THREADS)
k_direct_rows(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
              const uint8_t *__restrict__ types, int64_t n, int64_t nnz, int L,
              int64_t *__restrict__ ucount, uint64_t *__restrict__ sums, int64_t sum_words,
              uint64_t *__restrict__ counters, uint32_t *__restrict__ status) {
    __shared__ unsigned long long s_steps, s_deg;
    const int lane = lane_id();
    for (int64_t q = (int64_t)blockIdx.x * DIRECT_THREADS + threadIdx.x; q < sum_words;
         q += (int64_t)gridDim.x * DIRECT_THREADS)
        sums[q] = 0ull;
    if (threadIdx.x == 0) s_steps = s_deg = 0;
    __syncthreads();
    uint64_t steps = 0, most = 0;
    for (int64_t u = (int64_t)blockIdx.x * DIRECT_WAVES + threadIdx.x / WAVE; u < n;
         u += (int64_t)gridDim.x * DIRECT_WAVES) {
        const int64_t b = rp[u], e = rp[u + 1];
        uint32_t bad = 0;
        if (b < 0 || e > nnz || e < b || (u == 0 && b != 0) || (u == n - 1 && e != nnz)) {
            if (lane == 0) atomicOr(status, ST_UNSORTED);
            continue;
        }
        uint32_t up = 0;
        uint64_t near = 0;
        for (int64_t s = b + lane; s < e; s += WAVE) {
            const int32_t x = col[s];
            if (x == u) bad |= ST_SELF_LOOP;
            if (s > b && col[s - 1] >= x) bad |= ST_UNSORTED;
            if (x > u) ++up;
            if (x < 0 || x >= n) {
                bad |= ST_COL_RANGE;
                continue;
            }
            const int64_t xb = rp[x], xe = rp[x + 1];
            if (xb < 0 || xe > nnz || xe < xb) {
                bad |= ST_UNSORTED;
                continue;
            }
            near += (uint64_t)(xe - xb);
            const int64_t p = lower_bound(col, xb, xe, (int32_t)u);
            if (p >= xe || col[p] != (int32_t)u) bad |= ST_ASYMMETRIC;
        }
        near = wave_sum_u64(near);
        const uint64_t above = wave_sum_u64(up);
        bad = wave_or(bad);
        if (lane == 0) {
            if (types[u] >= L) bad |= ST_TYPE_RANGE;
            ucount[u] = (int64_t)above;
            if (bad) atomicOr(status, bad);
            steps += near * (uint64_t)(e - b);
            if ((uint64_t)(e - b) > most) most = (uint64_t)(e - b);
        }
    }
    if (lane == 0) {
        atomicAdd(&s_steps, (unsigned long long)steps);
        atomicMax(&s_deg, (unsigned long long)most);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_steps) atomicAdd((unsigned long long *)&counters[C_DIRECT_STEPS], s_steps);
        if (s_deg) atomicMax((unsigned long long *)&counters[C_DIRECT_DEG], s_deg);
    }
}

// One workgroup: first edge of every node, the edge count, and whether the
// walk is short enough (C_DIRECT_ON; the general pipeline runs otherwise).
__global__ void __launch_bounds__(1024)
k_direct_scan(const int64_t *__restrict__ ucount, int64_t n, int64_t m, uint32_t *__restrict__ eoff,
              uint64_t *__restrict__ counters, uint32_t *__restrict__ status) {
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x, lane = lane_id(), w = tid / WAVE;
    if (input_failed(status)) return;
    uint32_t carry = 0;
    for (int64_t q0 = 0; q0 < n; q0 += 1024) {
        const int64_t q = q0 + tid;
        const uint32_t c = q < n ? (uint32_t)ucount[q] : 0u;
        const uint32_t incl = wave_incl_scan(c);
        if (lane == WAVE - 1) wsum[w] = incl;
        __syncthreads();
        uint32_t add = carry, all = 0;
        for (int x = 0; x < 16; ++x) {
            if (x < w) add += wsum[x];
            all += wsum[x];
        }
        if (q < n) eoff[q] = add + incl - c;
        carry += all;
        __syncthreads();
    }
    if (tid == 0) {
        eoff[n] = carry;
        if ((int64_t)carry != m) atomicOr(status, ST_EDGE_COUNT);
        counters[C_DIRECT_ON] = counters[C_DIRECT_STEPS] <= DIRECT_STEPS &&
                                counters[C_DIRECT_DEG] <= (uint64_t)DIRECT_DEG;
    }
}

__host__ __device__ inline size_t direct_align(size_t x) { return (x + 15) & ~size_t(15); }

// Bytes of one wave's LDS: node marks, the near nodes, the orbit counts.
__host__ __device__ inline size_t direct_wave_lds(int64_t n, int L) {
    const int P = L * (L + 1) / 2;
    return direct_align((size_t)n) + direct_align(sizeof(uint16_t) * 2 * DIRECT_DEG) +
           direct_align(sizeof(uint32_t) * (size_t)(6 * P * ORBIT_COPIES + 3 * L)) +
           direct_align(sizeof(uint32_t) * 2 * WAVE);
}

// One wave per edge.  A node's byte in `mark` holds its type (bits 4-7) and,
// while an edge is counted, its membership in Gamma_u and Gamma_v (bits 0, 1).
// Bound by the latency of dependent row loads and by launches for small
// graphs, by the marks and counters in LDS for long walks.  The ER graph of
// 2,000 nodes and 8,000 edges took 379 us in the general pipeline (45
// launches) and takes 66 us, 100 edges 297 and 48 us.  Against the general
// pipeline with five types: 2^25 steps 255 and 565 us, 2^26.5 steps 482 and
// 697 us; beyond 2^27 steps the general pipeline is the faster.
__global__ void __launch_bounds__(WAVE * DIRECT_MOST)
k_direct_edges(const int64_t *__restrict__ rp, const int32_t *__restrict__ col,
               const uint8_t *__restrict__ types, int64_t n, int64_t m, int L,
               const uint32_t *__restrict__ eoff, uint64_t *__restrict__ rows, int gw, int hist_lds,
               uint64_t *__restrict__ sums, int copies, const uint64_t *__restrict__ counters,
               uint32_t *__restrict__ status) {
    extern __shared__ __align__(16) unsigned char sm_direct[];
    if (input_failed(status) || !counters[C_DIRECT_ON]) return;
    const int tid = threadIdx.x, lane = lane_id(), wv = tid / WAVE;
    const int waves = (int)blockDim.x / WAVE;
    const int P = L * (L + 1) / 2, W = 2 * L + 10 * P;
    const int n2 = (int)binom_small(L + 1, 2), n3 = (int)binom_small(L + 2, 3),
              n4 = (int)binom_small(L + 3, 4);
    uint64_t *gacc = sums + (size_t)(blockIdx.x % (unsigned)copies) * gw;
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(sm_direct);
    unsigned char *own = sm_direct + direct_align(hist_lds ? sizeof(uint64_t) * (size_t)gw : 0) +
                         (size_t)wv * direct_wave_lds(n, L);
    uint8_t *mark = own;
    uint16_t *near = reinterpret_cast<uint16_t *>(own + direct_align((size_t)n));
    uint32_t *acc = reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(near) +
                                                 direct_align(sizeof(uint16_t) * 2 * DIRECT_DEG));
    uint32_t *cls = acc + 6 * P * ORBIT_COPIES;   // |S_u^t|, |S_v^t|, |T^t|
    uint32_t *scan = reinterpret_cast<uint32_t *>(
        reinterpret_cast<unsigned char *>(acc) +
        direct_align(sizeof(uint32_t) * (size_t)(6 * P * ORBIT_COPIES + 3 * L)));
    uint32_t *first = scan + WAVE;   // first slot of each staged row
    auto gadd = [&](int idx, uint64_t v) {
        if (!v) return;
        if (hist_lds) atomicAdd(&hist[idx], (unsigned long long)v);
        else atomicAdd((unsigned long long *)&gacc[idx], (unsigned long long)v);
    };
    if (hist_lds)
        for (int q = tid; q < gw; q += (int)blockDim.x) hist[q] = 0ull;
    if (((uintptr_t)types & 3) == 0) {   // four types per load
        uint32_t *mark4 = reinterpret_cast<uint32_t *>(mark);
        const uint32_t *types4 = reinterpret_cast<const uint32_t *>(types);
#pragma unroll 4
        for (int64_t x = lane; x < n / 4; x += WAVE) mark4[x] = (types4[x] & 0x0f0f0f0fu) << 4;
        for (int64_t x = (n & ~int64_t(3)) + lane; x < n; x += WAVE) mark[x] = (uint8_t)(types[x] << 4);
    } else {
        for (int64_t x = lane; x < n; x += WAVE) mark[x] = (uint8_t)(types[x] << 4);
    }
    for (int q = lane; q < 6 * P * ORBIT_COPIES + 3 * L; q += WAVE) acc[q] = 0u;
    __syncthreads();
    uint32_t bad = 0;
    for (int64_t e = (int64_t)blockIdx.x * waves + wv; e < m;
         e += (int64_t)gridDim.x * waves) {
        // u: the last node whose first edge is at most e and which has edges,
        // found 64 candidates at a time
        int64_t lo = 0, hi = n;   // eoff[lo] <= e < eoff[hi]
        while (hi - lo > 1) {
            const int64_t step = (hi - lo + WAVE - 1) / WAVE;
            const int64_t q = lo + (lane + 1) * step;
            const bool in = q < hi && (int64_t)eoff[q] <= e;
            const int k = __popcll(__ballot(in));
            const int64_t nlo = lo + k * step, nhi = nlo + step;
            lo = nlo;
            if (nhi < hi) hi = nhi;
        }
        const int32_t u = (int32_t)lo;
        const int64_t ub = rp[u], ue = rp[u + 1];
        // u's entries above the diagonal are the last of its row
        const int32_t v = col[ue - (int64_t)(eoff[u + 1] - (uint32_t)e)];
        const int64_t vb = rp[v], ve = rp[v + 1];
        const int ta = types[u], tb = types[v];
        for (int64_t s = ub + lane; s < ue; s += WAVE) {
            const int32_t x = col[s];
            if (x != v) mark[x] |= 1;
        }
        wave_sync();
        // near nodes: Gamma_v without u, then Gamma_u without v and Gamma_v
        int nn = 0;
        for (int64_t s0 = vb; s0 < ve; s0 += WAVE) {
            const int64_t s = s0 + lane;
            const int32_t x = s < ve ? col[s] : u;
            const bool in = x != u;
            if (in) {
                const uint8_t c = mark[x];
                mark[x] = c | 2;
                atomicAdd(&cls[((c & 1) ? 2 : 1) * L + (c >> 4)], 1u);
            }
            const uint64_t bal = __ballot(in);
            if (in) near[nn + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)x;
            nn += __popcll(bal);
        }
        wave_sync();
        for (int64_t s0 = ub; s0 < ue; s0 += WAVE) {
            const int64_t s = s0 + lane;
            const int32_t x = s < ue ? col[s] : v;
            const uint8_t c = x != v ? mark[x] : 2;
            const bool in = (c & 2) == 0;
            if (in) atomicAdd(&cls[c >> 4], 1u);
            const uint64_t bal = __ballot(in);
            if (in) near[nn + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)x;
            nn += __popcll(bal);
        }
        wave_sync();
        // adjacent pairs {k, r}: orbit counter by the classes (1 S_u, 2 S_v,
        // 3 T, 0 neither) of k and r; pairs of two near nodes are met from
        // both ends and taken from one (fixed by class, else by id)
        for (int c0 = 0; c0 < nn; c0 += WAVE) {
            const int items = nn - c0 < WAVE ? nn - c0 : WAVE;
            uint32_t len = 0;
            if (lane < items) {
                const int64_t k = near[c0 + lane];
                const int64_t kb = rp[k];
                len = (uint32_t)(rp[k + 1] - kb);
                first[lane] = (uint32_t)kb;
            }
            const uint32_t incl = wave_incl_scan(len);
            scan[lane] = incl;
            const uint32_t total = __shfl(incl, WAVE - 1, WAVE);
            wave_sync();
            int o = 0;
            for (uint32_t f = lane; f < total; f += WAVE) {
                o = owner_next(scan, items, f, o);
                const int32_t k = near[c0 + o];
                const int32_t r = col[first[o] + (f - (o ? scan[o - 1] : 0u))];
                if (r == u || r == v) continue;
                const int mk = mark[k], mr = mark[r];
                const int ck = mk & 3, cr = mr & 3;
                // counters: 0 g3, 1 g8, 2 g6, 3 g7, 4 g10, 5 g12
                int z;
                if (cr == 0) z = ck == 3 ? 1 : 0;
                else if (ck == cr) z = k < r ? (ck == 3 ? 5 : 3) : -1;
                else if (ck == 3) z = 4;
                else z = ck == 1 && cr == 2 ? 2 : -1;
                if (z < 0) continue;
                int t = mk >> 4, w = mr >> 4;
                sort2(t, w);
                atomicAdd(&acc[(z * P + t * L - t * (t - 1) / 2 + (w - t)) * ORBIT_COPIES +
                               (lane & (ORBIT_COPIES - 1))],
                          1u);
            }
            wave_sync();
        }
        // the row and the global sums
        uint64_t *row = rows ? rows + (size_t)e * W : nullptr;
        if (lane == 0) gadd(rank2(ta, tb), 1);
        for (int t = lane; t < L; t += WAVE) {
            const uint64_t si = cls[t], sj = cls[L + t], tt = cls[2 * L + t];
            if (row) {
                row[t] = tt;
                row[L + t] = si + sj;
            }
            const int r3 = rank3(ta, tb, t);
            gadd(n2 + r3, si + sj);
            gadd(n2 + n3 + r3, tt);
        }
        for (int p = lane; p < P; p += WAVE) {
            int t = 0, rem = p;
            while (rem >= L - t) { rem -= L - t; ++t; }
            const int w = t + rem;
            const bool same = t == w;
            const int64_t at = cls[t], aw = cls[w], bt = cls[L + t], bw = cls[L + w],
                          ct = cls[2 * L + t], cw = cls[2 * L + w];
            auto orbit = [&](int z) {
                const uint32_t *c = acc + (z * P + p) * ORBIT_COPIES;
                uint32_t x = 0;
#pragma unroll
                for (int q = 0; q < ORBIT_COPIES; ++q) x += c[q];
                return (int64_t)x;
            };
            const int64_t g3 = orbit(0), g8 = orbit(1), g6 = orbit(2), g7 = orbit(3),
                          g10 = orbit(4), g12 = orbit(5);
            const int64_t g4 = (same ? at * bt : at * bw + aw * bt) - g6;                 // Lemma 1
            const int64_t g5 =
                (same ? at * (at - 1) / 2 + bt * (bt - 1) / 2 : at * aw + bt * bw) - g7;  // Lemma 2
            const int64_t g9 = (same ? ct * (at + bt) : ct * (aw + bw) + cw * (at + bt)) - g10;  // Lemma 3
            const int64_t g11 = (same ? ct * (ct - 1) / 2 : ct * cw) - g12;               // Lemma 4
            if (g4 < 0 || g5 < 0 || g9 < 0 || g11 < 0) bad |= ST_INTERNAL;
            if (row) {
                uint64_t *q = row + 2 * L + p;
                q[0] = (uint64_t)g3;
                q[P] = (uint64_t)g4;
                q[2 * P] = (uint64_t)g5;
                q[3 * P] = (uint64_t)g6;
                q[4 * P] = (uint64_t)g7;
                q[5 * P] = (uint64_t)g8;
                q[6 * P] = (uint64_t)g9;
                q[7 * P] = (uint64_t)g10;
                q[8 * P] = (uint64_t)g11;
                q[9 * P] = (uint64_t)g12;
            }
            const int h = n2 + 2 * n3 + rank4(ta, tb, t, w);
            gadd(h, (uint64_t)(g3 + g4));
            gadd(h + n4, (uint64_t)g5);
            gadd(h + 2 * n4, (uint64_t)g6);
            gadd(h + 3 * n4, (uint64_t)(g7 + g8 + g9));
            gadd(h + 4 * n4, (uint64_t)(g10 + g11));
            gadd(h + 5 * n4, (uint64_t)g12);
        }
        wave_sync();
        for (int q = lane; q < 6 * P * ORBIT_COPIES + 3 * L; q += WAVE) acc[q] = 0u;
        for (int q = lane; q < nn; q += WAVE) mark[near[q]] &= 0xf0;
        wave_sync();
    }
    bad = wave_or(bad);
    if (lane == 0 && bad) atomicOr(status, bad);
    __syncthreads();
    if (hist_lds)
        for (int q = tid; q < gw; q += (int)blockDim.x)
            if (hist[q]) atomicAdd((unsigned long long *)&gacc[q], hist[q]);
}

// The copies of the sums added up and divided by the graphlets' edge counts.
// A kernel of its own: a last-workgroup step inside the edge kernel needs a
// device-scope fence per workgroup, which writes the L2 back (60 of 85 us for
// the ER graph's 4 MB of rows).
__global__ void __launch_bounds__(256)
k_direct_finalize(const uint64_t *__restrict__ sums, int copies, int L, int gw,
                  uint64_t *__restrict__ global_counts, const uint64_t *__restrict__ counters,
                  uint32_t *__restrict__ status) {
    if (input_failed(status) || !counters[C_DIRECT_ON]) return;
    const int n2 = (int)binom_small(L + 1, 2), n3 = (int)binom_small(L + 2, 3),
              n4 = (int)binom_small(L + 3, 4);
    const uint64_t edges[9] = {1, 2, 3, 3, 3, 4, 4, 5, 6};
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= gw) return;
    int h;
    if (q < n2) h = 0;
    else if (q < n2 + n3) h = 1;
    else if (q < n2 + 2 * n3) h = 2;
    else h = 3 + (q - n2 - 2 * n3) / n4;
    uint64_t x = 0;
#pragma unroll 8
    for (int c = 0; c < copies; ++c) x += sums[(size_t)c * gw + q];
    if (x % edges[h]) atomicOr(status, ST_NOT_DIVISIBLE);
    global_counts[q] = x / edges[h];
}

bool direct_fits(int64_t n, int64_t m) {
    return n > 0 && n <= DIRECT_NODES && m <= DIRECT_EDGES;
}

hipError_t launch_direct(const int64_t *rp, const int32_t *col, const uint8_t *types, int64_t n,
                         int64_t nnz, int L, int gw, int64_t *ucount, uint32_t *eoff,
                         uint64_t *rows, uint64_t *sums, int64_t sum_words,
                         uint64_t *global_counts, uint64_t *counters, uint32_t *status, int cus, hipStream_t st) {
    const int64_t m = nnz / 2;
    int64_t copies = sum_words / gw;
    if (copies > DIRECT_COPIES) copies = DIRECT_COPIES;
    if (copies < 1) return hipErrorInvalidValue;
    int64_t grid = (n + DIRECT_WAVES - 1) / DIRECT_WAVES;
    if (grid > (int64_t)cus) grid = (int64_t)cus;
    k_direct_rows<<<(unsigned)grid, DIRECT_THREADS, 0, st>>>(rp, col, types, n, nnz, L, ucount,
                                                             sums, copies * gw, counters, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_direct_scan<<<1, 1024, 0, st>>>(ucount, n, m, eoff, counters, status);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int hist_lds = (size_t)gw * sizeof(uint64_t) <= 32768 ? 1 : 0;
    // one workgroup per CU of as many waves as its LDS holds: each workgroup
    // ends by adding its sums to a copy of the global ones
    const size_t head = direct_align(hist_lds ? (size_t)gw * sizeof(uint64_t) : 0);
    int64_t waves = (int64_t)((156 * 1024 - head) / direct_wave_lds(n, L));
    if (waves > DIRECT_MOST) waves = DIRECT_MOST;
    if (waves * cus > m) waves = (m + cus - 1) / cus;
    if (waves < 1) waves = 1;
    const size_t lds = head + (size_t)waves * direct_wave_lds(n, L);
    int64_t wgs = (m + waves - 1) / waves;
    if (wgs > cus) wgs = cus;
    if (wgs < 1) wgs = 1;
    k_direct_edges<<<(unsigned)wgs, (unsigned)(waves * WAVE), lds, st>>>(rp, col, types, n, m, L, eoff, rows,
                                                               gw, hist_lds, sums, (int)copies,
                                                               counters, status);
    e = hipGetLastError();
    if (e != hipSuccess || !global_counts) return e;
    k_direct_finalize<<<(unsigned)((gw + 255) / 256), 256, 0, st>>>(sums, (int)copies, L, gw,
                                                                    global_counts, counters, status);
    return hipGetLastError();
}

}  // namespace tg
