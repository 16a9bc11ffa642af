// Exclusive prefix sums over uint32 values: per-block sums, then a per-block scan
// that adds up the sums of the blocks before it itself; of more than
// kScanDirectBlocks blocks, a launch between the two scans the block sums.
// Load/Store are device functors, so a scan can gather its input and scatter
// its output (used for stream compaction and for the per-rank tile counts).
#pragma once
#include "common.hpp"

namespace mgs {

constexpr int kScanThreads = 256;
constexpr int kScanRounds = 8;
constexpr int kScanTile = kScanThreads * kScanRounds;  // 2048 values per block

// Exclusive scan of one value per thread across a 256-thread block.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *lds4, uint32_t *total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) lds4[wave] = x;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t s = lds4[w];
        before += (w < wave) ? s : 0u;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return before + x - v;
}

template <class Load>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(Load load, int64_t n, uint32_t *sums) {
    __shared__ uint32_t lds[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
#pragma unroll
    for (int r = 0; r < kScanRounds; ++r) {
        const int64_t i = base + r * kScanThreads + threadIdx.x;
        if (i < n) s += load(i);
    }
    uint32_t tot;
    block_exclusive_scan(s, lds, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// One block scans `nb` block sums in place; the grand total goes to *total.
static __global__ __launch_bounds__(kScanThreads) void k_scan_top(uint32_t *sums, int64_t nb, uint32_t *total) {
    __shared__ uint32_t lds[4];
    uint32_t carry = 0;
    for (int64_t base = 0; base < nb; base += kScanThreads) {
        const int64_t i = base + threadIdx.x;
        const uint32_t v = i < nb ? sums[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan(v, lds, &tot);
        if (i < nb) sums[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) {
        if (nb >= 0) sums[nb] = carry;
        if (total) *total = carry;
    }
}

// sum of v over the block, in every thread
__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t *lds4) {
    v = wave_sum_u32(v);
    if (lane_id() == 0) lds4[threadIdx.x >> 6] = v;
    __syncthreads();
    const uint32_t t = (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
    __syncthreads();
    return t;
}

// DIRECT: sums are the block sums (the last block also writes the grand total);
// else their exclusive scan.
template <class Load, class Store, bool DIRECT>
__global__ __launch_bounds__(kScanThreads) void k_scan_down(Load load, Store store, int64_t n,
                                                            const uint32_t *sums, uint32_t *total) {
    __shared__ uint32_t lds[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t carry = 0;
    if constexpr (DIRECT) {
        for (unsigned i = threadIdx.x; i < blockIdx.x; i += kScanThreads) carry += sums[i];
        carry = block_sum_u32(carry, lds);
    } else {
        carry = sums[blockIdx.x];
    }
    for (int r = 0; r < kScanRounds; ++r) {
        const int64_t i = base + r * kScanThreads + threadIdx.x;
        const uint32_t v = i < n ? load(i) : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan(v, lds, &tot);
        if (i < n) store(i, carry + ex, v);
        carry += tot;
    }
    if (DIRECT && total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = carry;
}

// A block of a direct scan reads up to this many sums, four a thread, from L2.
// The scan of 725 thousand values (354 blocks): 6.2 us for k_scan_down against
// 5.8 + 3.2 us for it and k_scan_top, and at every size one launch's gap less
// (3-6 us in a short chain).  The line lies where the mean read, half of this,
// would reach the top launch's cost by that slope (0.4 us for 354 sums).
constexpr int64_t kScanDirectBlocks = 1024;

inline int64_t scan_tmp_words(int64_t n) { return ceil_div(n, kScanTile) + 1; }

// tmp: at least scan_tmp_words(n) uint32; total: device uint32 (nullable).
template <class Load, class Store>
inline hipError_t scan_exclusive(Load load, Store store, int64_t n, uint32_t *tmp, uint32_t *total,
                                 hipStream_t s) {
    const int64_t nb = ceil_div(n, kScanTile);
    if (nb > 0) k_scan_reduce<Load><<<dim3((unsigned)nb), dim3(kScanThreads), 0, s>>>(load, n, tmp);
    if (nb > 0 && nb <= kScanDirectBlocks) {
        k_scan_down<Load, Store, true><<<dim3((unsigned)nb), dim3(kScanThreads), 0, s>>>(load, store, n, tmp, total);
        return hipGetLastError();
    }
    k_scan_top<<<1, kScanThreads, 0, s>>>(tmp, nb, total);
    if (nb > 0)
        k_scan_down<Load, Store, false><<<dim3((unsigned)nb), dim3(kScanThreads), 0, s>>>(load, store, n, tmp, nullptr);
    return hipGetLastError();
}

struct LoadU32 {
    const uint32_t *p;
    __device__ uint32_t operator()(int64_t i) const { return p[i]; }
};
struct StoreU32 {
    uint32_t *p;
    __device__ void operator()(int64_t i, uint32_t ex, uint32_t) const { p[i] = ex; }
};

// In-place scan of few values in one launch of one block (four a thread and
// round, all loads in flight), and their total.  p is 16-byte aligned.  Bound by
// the chain of load, wave scan and store: 4.4 us for 8 to 15 thousand values,
// against 3.6 + 5.3 us and a launch's gap for k_scan_reduce and k_scan_down.
constexpr int64_t kScanOneBlock = 16384;
static __global__ __launch_bounds__(1024) void k_scan_one(uint32_t *p, int n, uint32_t *total) {
    constexpr int kRounds = (int)(kScanOneBlock / 4096);
    __shared__ uint32_t sums[kRounds][16];
    const int i0 = 4 * (int)threadIdx.x, wave = (int)threadIdx.x >> 6;
    uint4 v[kRounds];
    uint32_t ex[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int i = 4096 * r + i0;
        if (i + 4 <= n) {
            v[r] = *reinterpret_cast<const uint4 *>(p + i);
        } else {
            v[r].x = i < n ? p[i] : 0u;
            v[r].y = i + 1 < n ? p[i + 1] : 0u;
            v[r].z = i + 2 < n ? p[i + 2] : 0u;
            v[r].w = 0u;
        }
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t sum = (v[r].x + v[r].y) + (v[r].z + v[r].w), incl = wave_incl_scan_u32(sum);
        ex[r] = incl - sum;
        if (lane_id() == 63) sums[r][wave] = incl;
    }
    __syncthreads();
    uint32_t carry = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        uint32_t o = carry + ex[r];
        for (int w = 0; w < 16; ++w) {
            o += w < wave ? sums[r][w] : 0u;
            carry += sums[r][w];
        }
        const uint4 e = make_uint4(o, o + v[r].x, o + v[r].x + v[r].y, o + v[r].x + v[r].y + v[r].z);
        const int i = 4096 * r + i0;
        if (i + 4 <= n) {
            *reinterpret_cast<uint4 *>(p + i) = e;
        } else {
            if (i < n) p[i] = e.x;
            if (i + 1 < n) p[i + 1] = e.y;
            if (i + 2 < n) p[i + 2] = e.z;
        }
    }
    if (threadIdx.x == 0) *total = carry;
}

}  // namespace mgs
