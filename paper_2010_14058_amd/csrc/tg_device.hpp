// Device helpers shared by the library's kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tg_internal.hpp"

namespace tg {

// ---------------------------------------------------------------- helpers

static __device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

static __device__ __forceinline__ int lane_id() { return threadIdx.x & (WAVE - 1); }

static __device__ __forceinline__ int64_t lower_bound(const int32_t *a, int64_t lo, int64_t hi,
                                               int32_t key) {
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

static __device__ __forceinline__ int64_t upper_bound(const int32_t *a, int64_t lo, int64_t hi,
                                               int32_t key) {
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] <= key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// First index in s[0..len) whose value exceeds f (s inclusive scan, LDS).
static __device__ __forceinline__ int owner_of(const uint32_t *s, int len, uint32_t f) {
    int lo = 0, hi = len;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (s[mid] <= f) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// owner_of for a thread whose item index f only grows: o is the owner of
// the previous f; most steps stay in the same item (one LDS read), else the
// search restarts above o.
static __device__ __forceinline__ int owner_next(const uint32_t *s, int len, uint32_t f, int o) {
    if (s[o] > f) return o;
    int lo = o + 1, hi = len;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (s[mid] <= f) lo = mid + 1; else hi = mid;
    }
    return lo;
}

static __device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    int lane = lane_id();
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        uint32_t o = __shfl_up(v, d, WAVE);
        if (lane >= d) v += o;
    }
    return v;
}

static __device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int d = WAVE / 2; d > 0; d >>= 1) v += (uint64_t)__shfl_xor((unsigned long long)v, d, WAVE);
    return v;
}

static __device__ __forceinline__ uint32_t wave_or(uint32_t v) {
#pragma unroll
    for (int d = WAVE / 2; d > 0; d >>= 1) v |= __shfl_xor(v, d, WAVE);
    return v;
}

static __device__ __forceinline__ uint32_t load_agent(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True once an input check has failed (the status word written by earlier
// kernels of the call): later kernels return at once.
static __device__ __forceinline__ bool input_failed(const uint32_t *status) {
    return (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ST_INPUT) != 0;
}

// The same for a check kernel whose workgroups meet at barriers: only the bits
// that it does not raise itself (`raised`) count.  Its other workgroups set
// those while it runs, and a wave that returned on one would leave the rest of
// its workgroup with shared memory that it should have filled.
static __device__ __forceinline__ bool failed_before(const uint32_t *status, uint32_t raised) {
    return (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ST_INPUT &
            ~raised) != 0;
}

// C(n, r) for r <= 4 (co-lexicographic ranks of type multisets).
static __device__ __forceinline__ int64_t binom_small(int64_t n, int r) {
    if (n < r) return 0;
    switch (r) {
        case 1: return n;
        case 2: return n * (n - 1) / 2;
        case 3: return n * (n - 1) * (n - 2) / 6;
        default: return n * (n - 1) * (n - 2) * (n - 3) / 24;
    }
}

static __device__ __forceinline__ void sort2(int &a, int &b) { if (a > b) { int c = a; a = b; b = c; } }

static __device__ __forceinline__ int rank2(int a, int b) {
    sort2(a, b);
    return (int)(binom_small(a, 1) + binom_small(b + 1, 2));
}

static __device__ __forceinline__ int rank3(int a, int b, int c) {
    sort2(a, b); sort2(b, c); sort2(a, b);
    return (int)(binom_small(a, 1) + binom_small(b + 1, 2) + binom_small(c + 2, 3));
}

static __device__ __forceinline__ int rank4(int a, int b, int c, int d) {
    sort2(a, b); sort2(c, d); sort2(a, c); sort2(b, d); sort2(b, c);
    return (int)(binom_small(a, 1) + binom_small(b + 1, 2) + binom_small(c + 2, 3) +
                 binom_small(d + 3, 4));
}

// Row offsets of the slots [s0, s1) one workgroup takes (flat over the CSR, so
// that a hub's row is spread over workgroups and short rows fill whole waves).
constexpr int SLOT_ROWS = 1024;

struct SlotTile {
    int64_t first[SLOT_ROWS + 1];   // offsets of rows r0 .. r1 + 1 when staged
    int64_t r0, r1;                 // rows holding the first and the last slot
    int staged;
};

// Smallest r with rp[r + 1] > key (rp nondecreasing, rp[n] > key), by a wave.
static __device__ __forceinline__ int64_t slot_search(const int64_t *rp, int64_t n, int64_t key) {
    int64_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int64_t step = (hi - lo + WAVE - 1) / WAVE;
        const int64_t q = lo + (lane_id() + 1) * step - 1;
        const int k = __popcll(__ballot(q < hi && rp[q + 1] <= key));
        lo += k * step;
        if (lo + step - 1 < hi) hi = lo + step - 1;
    }
    return lo;
}

// Fills T for slots [s0, s1), s0 < s1; by a whole workgroup of at least two waves.
static __device__ __forceinline__ void slot_tile(const int64_t *rp, int64_t n, int64_t s0,
                                                 int64_t s1, SlotTile &T) {
    const int w = threadIdx.x / WAVE;
    if (w < 2) {
        const int64_t r = slot_search(rp, n, w == 0 ? s0 : s1 - 1);
        if (lane_id() == 0) (w == 0 ? T.r0 : T.r1) = r;
    }
    __syncthreads();
    const int64_t rows = T.r1 - T.r0 + 1;
    if (threadIdx.x == 0) T.staged = rows <= SLOT_ROWS;
    if (rows <= SLOT_ROWS)
        for (int64_t q = threadIdx.x; q <= rows; q += blockDim.x) T.first[q] = rp[T.r0 + q];
    __syncthreads();
}

// First slot of row u of the tile (u up to r1 + 1).
static __device__ __forceinline__ int64_t slot_first(const int64_t *rp, const SlotTile &T, int64_t u) {
    return T.staged ? T.first[u - T.r0] : rp[u];
}

// Row of slot s, at least u (the row of an earlier slot of the same thread).
static __device__ __forceinline__ int64_t slot_row(const int64_t *rp, const SlotTile &T, int64_t u,
                                                   int64_t s) {
    if (slot_first(rp, T, u + 1) > s) return u;
    int64_t lo = u + 1, hi = T.r1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (slot_first(rp, T, mid + 1) <= s) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Super-hub bitmap probes: bit of node x in the bitmap of super-hub index s,
// and the slot of x inside the super-hub's (sorted) row.
static __device__ __forceinline__ bool sh_bit(const uint64_t *SB, int64_t nw, int s, int32_t x) {
    return (SB[(size_t)s * nw + (x >> 6)] >> (x & 63)) & 1ull;
}

static __device__ __forceinline__ int64_t sh_slot(const uint64_t *SB, const uint32_t *SP, int64_t nw,
                                                  int64_t row_begin, int s, int32_t x) {
    size_t o = (size_t)s * nw + (x >> 6);
    uint64_t below = (x & 63) ? (SB[o] & ((1ull << (x & 63)) - 1)) : 0ull;
    return row_begin + SP[o] + (uint32_t)__popcll(below);
}

}  // namespace tg
