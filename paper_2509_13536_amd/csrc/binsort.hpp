// Stable sort of the packed instance keys by their bin, in one counting pass
// over all bins, for calls whose bins' counters fit a block's LDS.  Four
// launches, of which the third also gives every bin's range of the list and the
// blend's work order:
//   k_binsort_hist     per block of consecutive instances: its count per bin
//   k_binsort_columns  per bin: exclusive scan of the blocks' counts, the total
//   k_bin_order        the bins' ranges from the totals, and the work order
//   k_binsort_scatter  each instance to its place
// In a scatter block each wave ranks its instances 64 at a time: ballots over
// the bin's bits find the lanes that share one, and the wave's counter of the
// bin in LDS carries the running rank, so equal bins keep the input order.
// The scatter is bound by its 8-byte writes, each to a line of its own (5.3M
// instances over 1200 bins 42 us, 6.9M over 3225 58 us); staging a block in bin
// order first, for whole runs, made 33 of the 42 but takes the LDS of a second
// block, and with twice the rows of counts gained nothing in sum.  Against two
// 8-bit radix passes and the search for the ranges, us: 62k instances over 300
// bins 24 -> 15, 5.3M over 1200 114 -> 61, 6.9M over 3225 137 -> 85.
#pragma once
#include "common.hpp"
#include "scan.hpp"

namespace mgs {

constexpr int kBinSortThreads = 512, kBinSortWaves = kBinSortThreads / 64;
// Counters of 16 bits, a row a wave, with the bin of unused slots.  Up to
// kBinSortFewBins they take 32 KB and the blocks' bases 8 KB, up to kBinSortMidBins
// twice that, two blocks on a CU.  Beyond, they are 104 KB, one block on a CU, whose
// bases no longer fit beside them and are gathered.  The time of a call's binning and
// sorting against that with radix passes: below 4096 bins 0.72 to 0.98 at every
// size from 500 to 49M instances.  Beyond, in calls of 2^17 to 2^22 instances: 4352 bins 0.88 to
// 0.97, 5400 0.91 to 0.99, 6450 0.92 to 0.99, 7500 0.97 to 1.04; of more, 4352 bins 0.95
// to 1.03, 6450 1.01 to 1.08, 8085 1.05 to 1.21.
constexpr int64_t kBinSortMaxBins = 6656, kBinSortManyMax = int64_t(1) << 22;
constexpr int kBinSortFewBins = 2048, kBinSortMidBins = 4096;
constexpr int kBinSortBits = 13;
static_assert(kBinSortMaxBins <= int64_t(1) << kBinSortBits, "a bin's bits");

// Rounds of 64 instances a wave takes: many where the table of counts (a row a
// block) has to stay small against the instances, few where the blocks have to
// fill the chip.  A call's binning and sorting at 2 / 8 / 16 rounds, us: 40k instances
// over 1200 bins 39 / 43 / 50, 260k 69 / 72 / 78, 917k 85 / 82 / 88; 2.9M over 3225
// bins - / 118 / 120, 4.6M over 1200 172 / 151 / 154, 12M over 3225 - / 257 / 261, 24M - / 471 / 440, 49M
// - / 880 / 816.  (2 rounds would serve up to 2^19, but leave no room for the table
// of 2048 bins and more.)
inline int binsort_rounds(int64_t m) { return m < (int64_t(1) << 17) ? 2 : m < (int64_t(1) << 24) ? 8 : 16; }
inline int64_t binsort_blocks(int64_t m) { return ceil_div(m, kBinSortThreads * binsort_rounds(m)); }
inline int64_t binsort_stride(int64_t bins) { return (bins + 1 + 63) / 64 * 64; }
// words of the table of counts, with the row of totals after it
inline int64_t binsort_words(int64_t m, int64_t bins) { return (binsort_blocks(m) + 1) * binsort_stride(bins); }
// Whether a call of m packed instances takes this sort.  The table has to fit
// `room` words, the value arrays that such keys leave unused, about 2 m: from 2^17
// instances on it does at any of these bins, below them up to 1983 bins (128
// words for 64 instances, 31 thousand instances at 1983 bins).
inline bool binsort_takes(int64_t m, int64_t bins, int64_t room) {
    if (m <= 0 || bins >= kBinSortMaxBins || (bins >= kBinSortMidBins && m >= kBinSortManyMax)) return false;
    if (binsort_rounds(m) == 2 && binsort_stride(bins) > kBinSortFewBins) return false;
    return binsort_words(m, bins) <= room;
}

// bin of a key: unused slots hold all ones there and count as bin n_bins
__device__ __forceinline__ uint32_t binsort_bin(uint32_t low, uint32_t mask, uint32_t n_bins) {
    return min(low & mask, n_bins);
}

// Consecutive blocks go to the eight XCDs in turn; their L2s are apart.  Block b
// takes part such that one XCD's blocks hold consecutive instances, whose places
// in a bin's list are consecutive too: its L2 then fills the lines it writes.
__device__ __forceinline__ int64_t binsort_part(int64_t b, int64_t nb) {
    const int64_t q = nb >> 3, r = nb & 7, x = b & 7;
    return x * q + min(x, r) + (b >> 3);
}

template <int ROUNDS, int BINS>
__global__ __launch_bounds__(kBinSortThreads) void k_binsort_hist(const uint64_t *keys, int64_t m, uint32_t mask,
                                                                  uint32_t n_bins, int stride, uint32_t *table) {
    __shared__ uint32_t h[BINS];
    const int64_t part = binsort_part(blockIdx.x, gridDim.x);
    const int64_t base = part * (kBinSortThreads * ROUNDS) + threadIdx.x;
    uint32_t low[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = base + r * kBinSortThreads;
        low[r] = i < m ? reinterpret_cast<const uint32_t *>(keys)[2 * i] : 0u;
    }
    for (int i = (int)threadIdx.x; i < stride; i += kBinSortThreads) h[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
        if (base + r * kBinSortThreads < m) atomicAdd(&h[binsort_bin(low[r], mask, n_bins)], 1u);
    __syncthreads();
    for (int i = (int)threadIdx.x; i < stride; i += kBinSortThreads) table[part * stride + i] = h[i];
}

// 32 bins a block; each of its 32 half-waves scans a run of the blocks' rows.
__global__ __launch_bounds__(1024) void k_binsort_columns(uint32_t *table, int64_t nb, int stride) {
    __shared__ uint32_t sums[32][33];
    const int c = (int)threadIdx.x & 31, part = (int)threadIdx.x >> 5;
    uint32_t *col = table + (int64_t)blockIdx.x * 32 + c;
    const int64_t per = (nb + 31) / 32, r0 = min(part * per, nb), r1 = min(r0 + per, nb);
    uint32_t sum = 0;
    constexpr int kAhead = 8;
    for (int64_t r = r0; r < r1; r += kAhead) {
        uint32_t v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = r + u < r1 ? col[(r + u) * stride] : 0u;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) sum += v[u];
    }
    sums[part][c] = sum;
    __syncthreads();
    uint32_t ex = 0;
    for (int p = 0; p < part; ++p) ex += sums[p][c];
    if (part == 31) col[nb * stride] = ex + sum;
    for (int64_t r = r0; r < r1; r += kAhead) {
        uint32_t v[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = r + u < r1 ? col[(r + u) * stride] : 0u;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (r + u < r1) col[(r + u) * stride] = ex;
            ex += v[u];
        }
    }
}

template <int ROUNDS, int BINS>
__global__ __launch_bounds__(kBinSortThreads) void k_binsort_scatter(const uint64_t *keys, uint64_t *out, int64_t m,
                                                                     uint32_t mask, int bits, uint32_t n_bins,
                                                                     int stride, const uint32_t *table,
                                                                     const uint2 *range) {
    __shared__ uint32_t cnt32[kBinSortWaves][BINS / 2];  // two 16-bit counters a word
    constexpr bool kBases = BINS <= kBinSortMidBins;  // the bases in LDS, else gathered
    __shared__ uint32_t gbase[kBases ? BINS : 1];
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t part = binsort_part(blockIdx.x, gridDim.x);
    const int64_t base = part * (kBinSortThreads * ROUNDS) + wave * (64 * ROUNDS) + lane;
    uint64_t key[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) key[r] = base + 64 * r < m ? keys[base + 64 * r] : 0ull;
    const int words = stride / 2;
    for (int w = 0; w < kBinSortWaves; ++w)
        for (int i = (int)threadIdx.x; i < words; i += kBinSortThreads) cnt32[w][i] = 0u;
    __syncthreads();
    typedef uint16_t __attribute__((may_alias)) Count;
    Count *cnt = reinterpret_cast<Count *>(cnt32[wave]);
    const uint64_t lt = (1ull << lane) - 1ull;
    uint32_t rank[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const bool valid = base + 64 * r < m;
        const uint32_t d = binsort_bin((uint32_t)key[r], mask, n_bins);
        const uint64_t in = ballot(valid);
        uint32_t plo = (uint32_t)in, phi = (uint32_t)(in >> 32);
#pragma unroll
        for (int b = 0; b < kBinSortBits; ++b) {
            if (b >= bits) break;  // uniform
            const int same = (int)(d << (31 - b)) >> 31;  // the bit in every position
            const uint64_t s = ballot(same != 0);
            plo &= ~((uint32_t)s ^ (uint32_t)same);
            phi &= ~((uint32_t)(s >> 32) ^ (uint32_t)same);
        }
        const uint64_t peers = (uint64_t)phi << 32 | plo;
        const uint32_t before = cnt[d];
        wave_lds_sync();
        rank[r] = before + (uint32_t)__popcll(peers & lt);
        if (valid && (peers & ~lt) >> lane == 1ull) cnt[d] = (Count)(rank[r] + 1u);  // the last of its bin
        wave_lds_sync();
    }
    __syncthreads();
    // where the block's part of each bin begins, and each wave's in it
    for (int i = (int)threadIdx.x; i < words; i += kBinSortThreads) {
        uint32_t ex = 0;
#pragma unroll
        for (int w = 0; w < kBinSortWaves; ++w) {
            const uint32_t c = cnt32[w][i];
            cnt32[w][i] = ex;
            ex += c;  // both halves: a block holds fewer than 2^16 instances
        }
        if (!kBases) continue;
        const uint2 t = *reinterpret_cast<const uint2 *>(table + part * stride + 2 * i);
        gbase[2 * i] = 2 * i <= (int)n_bins ? range[2 * i].x + t.x : 0u;
        gbase[2 * i + 1] = 2 * i + 1 <= (int)n_bins ? range[2 * i + 1].x + t.y : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        if (base + 64 * r >= m) continue;
        const uint32_t d = binsort_bin((uint32_t)key[r], mask, n_bins);
        const uint32_t at = kBases ? gbase[d] : range[d].x + table[part * stride + d];
        out[at + cnt[d] + rank[r]] = key[r];
    }
}

}  // namespace mgs
