// Mapping loss of MemGS (Sec. II-E, Eq. (12)) for gfx950: colour L1, SSIM,
// masked depth L1 and the isotropy term L_iso, value and gradient.
//
//   k_loss        one launch.  Blocks of SSIM tiles: value and gradient of the
//                 SSIM and L1 terms of a strip of one colour channel, in one pass
//                 over the images.  Blocks of the depth residual and its
//                 gradient.  Blocks of L_iso, in fp64, so that the sign of each
//                 scale's deviation from the mean scale is decided exactly.
//   k_loss_put    only where the colour gradient overlaps an image: copies it there
//   k_loss_final  one block: fixed-order fp64 sums of the blocks' partial sums (of
//                 many views k_loss_views before it), then the total in view
//                 order, so the values are deterministic.
//
// The colour terms move 8 bytes in and 4 out per pixel and channel.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

#include "api_range.hpp"
#include "common.hpp"

namespace mgs {
namespace {

constexpr int kLR = 5;              // window radius
constexpr int kLW = 2 * kLR + 1;    // window taps
constexpr float kC1 = 1e-4f;        // (0.01)^2
constexpr float kC2 = 9e-4f;        // (0.03)^2

struct LossView {
    int32_t W, H;
    int32_t strips;      // strips of kSC columns
    int32_t tile_base;   // first SSIM tile of the view (strips of one channel, cut into segments of rows)
    int64_t pix_base;    // first pixel in the packed one-channel layout
    int32_t depth_base;  // first block of the depth residual
    float inv_n3;        // 1 / (3 W H)
    float inv_n1;        // 1 / (W H)
    int32_t pad;
};
// The table of 89 views fits the arguments of k_arg_copy, and its size is a part
// of the workspace that the entry points ask for.
static_assert(sizeof(LossView) == 40 && 89 * sizeof(LossView) <= 4 * (size_t)kArgCopyWords, "view table");

// A call of at most kArgViews views carries its view table in the kernel
// arguments; a larger one copies it to the workspace.
constexpr int kArgViews = 16;
struct ViewTable {
    const LossView *table;  // null: the views are in own
    LossView own[kArgViews];
    int32_t n;
    __device__ __forceinline__ const LossView &operator[](int v) const { return table ? table[v] : own[v]; }
};

struct SsimArgs {
    ViewTable views;
    int64_t n_tiles;  // per channel
    int nch;          // column chunks of a tile
    const float *rgb, *gt;
    float *partial;   // [3][n_tiles][2]: sum of 1 - SSIM, of |x - y|
    float *d_rgb;
    float lam;
    float w[kLW];     // normalised window weights
};

__device__ __forceinline__ float sgnf(float d) { return d > 0.0f ? 1.0f : (d < 0.0f ? -1.0f : 0.0f); }

// ---------------------------------------------------------------- colour: SSIM and L1
// A block of four waves takes a strip of 54 output columns of one channel and
// marches down its rows in chunks of 8.  The window is needed twice: over the
// moments E[x], E[y], E[(x - y)^2], E[xy] (the variances enter only as their
// sum) and over the three derivative maps.  Both filters are carried along the
// march, so the maps never leave the chip: memory sees x and y once (their halo
// again through the caches) and the gradient.
//
// The two windows are 154 FMAs per pixel and channel, 50 us on 8 x 1200 x 680 at the
// rate the vector units reach (2.6 cycles an FMA on a SIMD with vector operands
// alone, 4.4 with a scalar one: the weights are kept in vector registers).  x, y and
// the gradient are 235 MB there, 50 us.  It takes 175 us, where two kernels with the
// maps in memory between them took 348.  With the halo, the rows of warm-up, the
// formula and the transposes a pixel and channel take 316 lane instructions, 97M of a
// wave: about 130 us of issue at those rates; the LDS is busy 82 us, a quarter of it
// with bank conflicts, and the waves wait for it and at three barriers a chunk.  One wave for all signals of a strip carries 84
// sums a lane and leaves two waves to a SIMD, which wait for each other's
// memory: 174 us without the depth residual, and slower in a call of one view,
// whose time is that of a chunk.  A wave for each signal carries 24.
//
//   A  wave w: signal w of the chunk's 8 rows (lanes = 8 rows x 8 bands of 8 map
//      columns, 18 input columns a lane), filtered along x; transposed through
//      LDS (lanes = the 64 map columns); along y, four rows at a time, the sums
//      of the 12 rows in progress kept in registers
//   B  wave t: SSIM and its derivatives of two of the eight complete map rows
//   C  wave k < 3: map k along y; transposed (lanes = 8 rows x 8 bands of 8
//      columns, of which 54 are output); along x
//      then, a wave two rows, the gradient
//
// A map row completes three quads of rows after its first input, an output row
// another three: chunk j completes map rows 8 j - 12 .. - 5 and output rows
// 8 j - 24 .. - 17 of the tile, which has 8 nch - 24 output rows.
constexpr int kSC = 54;               // output columns of a strip
constexpr int kWarm = 24;             // rows of warm-up of a tile
constexpr int kIn = 8 + 2 * kLR;      // inputs of a band of 8 outputs along x
constexpr int kInC = 64 + 2 * kLR;    // input columns of a strip
constexpr int kStage = (8 * kInC + 255) / 256;  // staged values of a thread and image
static_assert(kSC + 2 * kLR == 64, "the lane layouts");
// LDS of one signal, in the row layout (row r at row_at(r)) or the column layout
// (column c at 12 c): the 16-byte reads of a band's row, and those of a
// column's rows, then meet no bank twice.
constexpr int kSig = 768, kRows = 648;
__device__ __forceinline__ constexpr int row_at(int r) { return 80 * r + 4 * (r >> 2); }
static_assert(kInC <= 80 && row_at(7) + 80 <= kRows && 12 * 63 + 8 <= kSig, "LDS of a signal");

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));

template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

__device__ __forceinline__ int uniform_i(int x) { return __builtin_amdgcn_readfirstlane(x); }

// acc[m] += w[K - m] v for a group's four outputs
template <int K>
__device__ __forceinline__ void mac4(const float *w, float v, f4 &acc) {
#pragma unroll
    for (int m = 0; m < 4; ++m)
        if (K - m >= 0 && K - m < kLW) acc[m] = __builtin_fmaf(w[K - m], v, acc[m]);
}

// Filtering along y: four new rows into the three groups of four outputs in
// progress (oldest first) and a new one; the oldest completes.
__device__ __forceinline__ f4 next_quad(const float *w, f4 in, f4 (&g)[3]) {
    f4 n = {0.0f, 0.0f, 0.0f, 0.0f};
    mac4<12>(w, in[0], g[0]);
    mac4<13>(w, in[1], g[0]);
    static_for<4>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        mac4<8 + c>(w, in[c], g[1]);
        mac4<4 + c>(w, in[c], g[2]);
        mac4<c>(w, in[c], n);
    });
    const f4 done = g[0];
    g[0] = g[1];
    g[1] = g[2];
    g[2] = n;
    return done;
}

__device__ __forceinline__ float plane_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

// A band's eight outputs along x from its row at p; get(k): inputs 4 k .. 4 k + 3.
// One quad of inputs at a time, which keeps the registers few.
template <class F>
__device__ __forceinline__ void filter_band(const float *w, F &&get, f4 (&v)[2]) {
    v[0] = v[1] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    static_for<5>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        const f4 x = get(kc);
#pragma unroll
        for (int i = 0; i < (k < 4 ? 4 : 2); ++i)
#pragma unroll
            for (int o = 0; o < 8; ++o)
                if (4 * k + i - o >= 0 && 4 * k + i - o < kLW)
                    v[o >> 2][o & 3] = __builtin_fmaf(w[4 * k + i - o], x[i], v[o >> 2][o & 3]);
        __builtin_amdgcn_sched_barrier(0);
    });
}

// One tile of one channel: item = channel * n_tiles + tile.
__device__ __forceinline__ void ssim_tile(const SsimArgs &a, int64_t item) {
    __shared__ __attribute__((aligned(16))) float mom[4][kSig], map[3][kSig], img[2][kRows];
    __shared__ float red[2][4];
    const int c = (int)(item / a.n_tiles);
    const int64_t tile = item - c * a.n_tiles;
    int lo = 0, hi = a.views.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.views[mid].tile_base <= tile) lo = mid; else hi = mid - 1;
    }
    const LossView &V = a.views[lo];
    // scalars (the view's address may be in either memory, so the compiler
    // would take what it loads for a lane's own)
    const int W = uniform_i(V.W), H = uniform_i(V.H), strips = uniform_i(V.strips);
    const int64_t pix_base = (int64_t)(uint32_t)uniform_i((int)V.pix_base) | ((int64_t)uniform_i((int)(V.pix_base >> 32)) << 32);
    const float inv_n3 = V.inv_n3;
    const int lt = uniform_i((int)(tile - V.tile_base)), sg = lt / strips;
    const int c0 = (lt - sg * strips) * kSC, r0 = sg * (8 * a.nch - kWarm);
    const int rend = min(r0 + 8 * a.nch - kWarm, H);  // output rows [r0, rend)
    const int lane = lane_id(), w = uniform_i((int)threadIdx.x >> 6);
    const int band = lane >> 3, row = lane & 7;
    const int64_t plane = (int64_t)W * H, cbase = 3 * pix_base + c * plane;
    // rows and columns outside the image read as zero: their offset is one past
    // the plane
    const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.rgb + cbase), (short)0, (int)(4 * plane), 0x00027000);
    const auto ry = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.gt + cbase), (short)0, (int)(4 * plane), 0x00027000);
    constexpr uint32_t kOutside = 0x80000000u;
    const uint32_t pitch = 4u * (uint32_t)W;
    const int map_col = c0 - kLR + lane;              // this lane's map column in the column layout
    const bool col_in = map_col >= 0 && map_col < W;
    const bool col_own = col_in && lane >= kLR && lane < kLR + kSC;
    const int ox = c0 + lane;                         // and its output column
    const bool out_own = lane < kSC && ox < W;
    const int at_col = 12 * lane;                     // its place in the column layout
    const int at_band = row_at(row) + 8 * band;       // this lane's band of 8 in the row layout
    const float kl1 = (1.0f - a.lam) * inv_n3, ks = 2.0f * (a.lam * inv_n3);  // the maps are halves
    const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f4 g1[3] = {zero, zero, zero}, g2[3] = {zero, zero, zero};
    // the weights in vector registers: an FMA with a scalar operand issues at
    // about half the rate
    float wv[kLW];
#pragma unroll
    for (int o = 0; o <= kLR; ++o) {
        float t = a.w[o];
        asm volatile("" : "+v"(t));
        wv[o] = wv[kLW - 1 - o] = t;
    }
    float sS = 0.0f, sL = 0.0f;
    float xo[2], yo[2];  // x and y of this wave's two output rows
    // staging of a chunk's 8 x 74 values of both images: loaded a chunk ahead
    float xs[kStage], ys[kStage];
    uint32_t soff[kStage];
    int slds[kStage];
#pragma unroll
    for (int k = 0; k < kStage; ++k) {
        const int i = (int)threadIdx.x + 256 * k, r = i / kInC, q = i - r * kInC, gx = c0 - 2 * kLR + q;
        const bool in = r < 8 && gx >= 0 && gx < W;
        soff[k] = in ? (uint32_t)(r0 - 2 * kLR + r) * pitch + 4u * (uint32_t)gx : kOutside;
        slds[k] = r < 8 ? row_at(r) + q : kInC;  // a spare place
    }
    auto stage_load = [&]() {
#pragma unroll
        for (int k = 0; k < kStage; ++k) {
            xs[k] = plane_load(rx, soff[k]);
            ys[k] = plane_load(ry, soff[k]);
            soff[k] += 8 * pitch;
        }
    };
    auto stage_store = [&]() {
#pragma unroll
        for (int k = 0; k < kStage; ++k) {
            img[0][slds[k]] = xs[k];
            img[1][slds[k]] = ys[k];
        }
    };
    stage_load();
    stage_store();
    stage_load();
    __syncthreads();
    float *const my = mom[w];
    // the gradient of the 8 rows from gy0 on, from the maps' sums in LDS
    auto finish = [&](int gy0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = 2 * w + u, oy = gy0 + r;  // uniform
            if (oy >= rend) break;
            if (out_own) {
                const float o0 = map[0][row_at(r) + lane], o1 = map[1][row_at(r) + lane], o2 = map[2][row_at(r) + lane];
                const float d = xo[u] - yo[u];
                const float gs = o0 + (xo[u] * o1 + yo[u] * o2);  // no FMA: 0 of equal images
                a.d_rgb[cbase + (int64_t)oy * W + ox] = __builtin_fmaf(-ks, gs, kl1 * sgnf(d));
                sL += fabsf(d);
            }
        }
    };
    for (int j = 0; j < a.nch; ++j) {
        // A
        {
            if (j > 3) finish(r0 + 8 * (j - 1) - kWarm);
            f4 v[2];
            const float *const x = img[0] + at_band, *const y = img[1] + at_band;
            auto quad = [](const float *p, auto kc) { return *reinterpret_cast<const f4 *>(p + 4 * decltype(kc)::value); };
            if (w < 2) {
                const float *const p = w == 0 ? x : y;
                filter_band(wv, [&](auto kc) { return quad(p, kc); }, v);
            } else if (w == 2) {
                filter_band(wv, [&](auto kc) {
                    const f4 p = quad(x, kc), q = quad(y, kc);
                    f4 e;
#pragma unroll
                    for (int i = 0; i < 4; ++i) e[i] = (p[i] - q[i]) * (p[i] - q[i]);
                    return e;
                }, v);
            } else {
                filter_band(wv, [&](auto kc) { return quad(x, kc) * quad(y, kc); }, v);
            }
            *reinterpret_cast<f4 *>(my + at_band) = v[0];
            *reinterpret_cast<f4 *>(my + at_band + 4) = v[1];
            wave_lds_sync();
            f4 q0, q1;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                q0[r] = my[row_at(r) + lane];
                q1[r] = my[row_at(r + 4) + lane];
            }
            wave_lds_sync();
            const f4 d0 = next_quad(wv, q0, g1), d1 = next_quad(wv, q1, g1);
            *reinterpret_cast<f4 *>(my + at_col) = d0;
            *reinterpret_cast<f4 *>(my + at_col + 4) = d1;
        }
        __syncthreads();
        // B
        stage_store();
        stage_load();
        {
            const f2 mx2 = *reinterpret_cast<const f2 *>(mom[0] + at_col + 2 * w), my2 = *reinterpret_cast<const f2 *>(mom[1] + at_col + 2 * w);
            const f2 e2 = *reinterpret_cast<const f2 *>(mom[2] + at_col + 2 * w), p2 = *reinterpret_cast<const f2 *>(mom[3] + at_col + 2 * w);
            f2 M[3];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int gy = r0 - kLR + 8 * j - 12 + 2 * w + u;  // uniform
                const bool in = col_in && gy >= 0 && gy < H;
                const float mx = mx2[u], my = my2[u], e = e2[u], p = p2[u];
                // SSIM = (1 - a) (1 - b), a and b differences of the two images over sums,
                // so that equal windows give 1, no derivative by E[x], and those by E[x^2]
                // (twice it) and E[xy] opposite, exactly; 1 - SSIM keeps its small values.
                // The maps hold half of each
                const float dm = mx - my, dd = dm * dm, ed = e - dd;
                const float iC = __builtin_amdgcn_rcpf(__builtin_fmaf(mx, mx, my * my) + kC1);
                const float iD = __builtin_amdgcn_rcpf(__builtin_fmaf(2.0f, __builtin_fmaf(-mx, my, p), ed) + kC2);
                const float a1 = dd * iC, b1 = ed * iD, u1 = 1.0f - a1, v1 = 1.0f - b1, uD = u1 * iD;
                const float d0 = __builtin_fmaf(v1 * iC, __builtin_fmaf(-mx, u1, my), uD * __builtin_fmaf(mx, v1, -my));
                M[0][u] = in ? d0 : 0.0f;
                M[1][u] = in ? -uD * v1 : 0.0f;
                M[2][u] = in ? uD : 0.0f;
                if (gy >= r0 && gy < rend) sS += col_own ? __builtin_fmaf(-a1, b1, a1 + b1) : 0.0f;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) *reinterpret_cast<f2 *>(map[k] + at_col + 2 * w) = M[k];
        }
        __syncthreads();
        // C
        if (j >= 3) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int oy = r0 + 8 * j - kWarm + 2 * w + u;
                const uint32_t off = out_own && oy < H ? (uint32_t)oy * pitch + 4u * (uint32_t)ox : kOutside;
                xo[u] = plane_load(rx, off);
                yo[u] = plane_load(ry, off);
            }
        }
        if (w < 3) {
            float *const mp = map[w];
            const f4 q0 = *reinterpret_cast<const f4 *>(mp + at_col), q1 = *reinterpret_cast<const f4 *>(mp + at_col + 4);
            wave_lds_sync();
            const f4 d0 = next_quad(wv, q0, g2), d1 = next_quad(wv, q1, g2);
            if (j >= 3) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    mp[row_at(r) + lane] = d0[r];
                    mp[row_at(r + 4) + lane] = d1[r];
                }
                wave_lds_sync();
                f4 v[2];
                filter_band(wv, [&](auto kc) { return *reinterpret_cast<const f4 *>(mp + at_band + 4 * decltype(kc)::value); }, v);
                wave_lds_sync();
                *reinterpret_cast<f4 *>(mp + at_band) = v[0];
                *reinterpret_cast<f4 *>(mp + at_band + 4) = v[1];
            }
        }
        __syncthreads();
    }
    finish(r0 + 8 * (a.nch - 1) - kWarm);
    sS = wave_sum(sS);
    sL = wave_sum(sL);
    if (lane == 0) {
        red[0][w] = sS;
        red[1][w] = sL;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        *reinterpret_cast<float2 *>(a.partial + 2 * item) =
            make_float2((red[0][0] + red[0][1]) + (red[0][2] + red[0][3]), (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]));
}

__device__ __forceinline__ double sgnd(double d) { return d > 0.0 ? 1.0 : (d < 0.0 ? -1.0 : 0.0); }

__device__ __forceinline__ double wave_sum_f64(double x) {
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

// ---------------------------------------------------------------- depth and L_iso
constexpr int kDepthPix = 8192;  // pixels of one view that a block takes
constexpr int kIsoGauss = 1024;  // Gaussians that a block of L_iso takes

struct RestArgs {
    int64_t n_depth;  // blocks of the depth residual
    const float *depth, *gtd;
    float *d_depth, *depth_partial;
    float w_depth;
    const float *scales;
    int64_t n;
    float w_iso;
    float *d_scales;
    double *iso_partial;
};

__device__ __forceinline__ void depth_block(const RestArgs &a, const ViewTable &views, int64_t b) {
    __shared__ float red[4];
    int lo = 0, hi = views.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].depth_base <= b) lo = mid; else hi = mid - 1;
    }
    const LossView &V = views[lo];
    const int64_t n = (int64_t)V.W * V.H, base = (b - V.depth_base) * kDepthPix;
    const float *D = a.depth + V.pix_base, *G = a.gtd + V.pix_base;
    const float k = a.w_depth * V.inv_n1;
    float sum = 0.0f;
    for (int64_t i0 = base + threadIdx.x; i0 < base + kDepthPix; i0 += 256 * 8) {
        float d[8], g[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t i = i0 + 256 * r;
            d[r] = i < n ? D[i] : 0.0f;
            g[r] = i < n ? G[i] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const float e = g[r] > 0.0f ? d[r] - g[r] : 0.0f;
            sum += fabsf(e);
            if (i0 + 256 * r < n) a.d_depth[V.pix_base + i0 + 256 * r] = k * sgnf(e);
        }
    }
    sum = wave_sum(sum);
    if (lane_id() == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) a.depth_partial[b] = (red[0] + red[1]) + (red[2] + red[3]);
}

// deviations of the Gaussians' three scales from their mean
__device__ __forceinline__ void iso_block(const RestArgs &a, int64_t b) {
    __shared__ double red[4];
    double acc = 0.0;
    const double k = (double)a.w_iso / (3.0 * (double)a.n);
    for (int64_t g = b * kIsoGauss + threadIdx.x; g < std::min<int64_t>(a.n, (b + 1) * kIsoGauss); g += 256) {
        const double s0 = a.scales[3 * g], s1 = a.scales[3 * g + 1], s2 = a.scales[3 * g + 2];
        const double m = (s0 + s1 + s2) / 3.0;
        const double e0 = s0 - m, e1 = s1 - m, e2 = s2 - m;
        acc += fabs(e0) + fabs(e1) + fabs(e2);
        const double g0 = sgnd(e0), g1 = sgnd(e1), g2 = sgnd(e2);
        const double mg = (g0 + g1 + g2) / 3.0;
        a.d_scales[3 * g] = (float)(k * (g0 - mg));
        a.d_scales[3 * g + 1] = (float)(k * (g1 - mg));
        a.d_scales[3 * g + 2] = (float)(k * (g2 - mg));
    }
    acc = wave_sum_f64(acc);
    if (lane_id() == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) a.iso_partial[b] = red[0] + red[1] + red[2] + red[3];
}

// The whole loss but its sums, in one launch: the SSIM tiles, which issue is the
// bound of, then blocks of the depth residual and of L_iso, which memory is, in
// the room that the last tiles leave.  Workgroups are dealt to the eight XCDs
// round robin (block b on XCD b % 8); each XCD gets a contiguous run of tiles, so
// the halo a tile shares with its neighbours is read through the same L2.  The
// tiles have 8 ceil(n / 8) blocks; those past the last tile exit.
__global__ __launch_bounds__(256, 5) void k_loss(SsimArgs a, RestArgs r) {
    const int64_t n = 3 * a.n_tiles, per = (n + 7) / 8, b = blockIdx.x;
    if (b < 8 * per) {
        const int64_t item = (b & 7) * per + (b >> 3);
        if (item < n) ssim_tile(a, item);
    } else if (b - 8 * per < r.n_depth) {
        depth_block(r, a.views, b - 8 * per);
    } else {
        iso_block(r, b - 8 * per - r.n_depth);
    }
}

// The colour gradient of a call whose dL_drgb overlaps an image.  A tile reads its
// neighbours' pixels, so k_loss leaves the gradient in the workspace there.
__global__ __launch_bounds__(256) void k_loss_put(const float *from, float *to, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) to[i] = from[i];
}

// ---------------------------------------------------------------- values
struct FinalArgs {
    ViewTable views;
    int64_t n_tiles, n_depth;
    const float *partial, *depth_partial;
    const double *iso_partial;
    int64_t n_iso_blocks;
    int64_t n_gauss;
    float lam, w_depth, w_iso;
    int has_depth;
    double *terms;  // [n_views]: L_view of each view, of more than kArgViews
    float *loss;    // [4 n_views + 2]
};

// Terms of views v0 .. v0 + at_once - 1, by 16 waves, `share` to a view, summed in
// a fixed order.  out: [at_once] L_view.
__device__ __forceinline__ void view_terms(const FinalArgs &a, int v0, int at_once, int share, double *out) {
    __shared__ double red[3][16];
    const int lane = lane_id(), wave = threadIdx.x >> 6, nv = a.views.n, v = v0 + wave / share;
    double sS = 0.0, sL = 0.0, sD = 0.0;
    if (wave < at_once * share && v < nv) {
        const int64_t t0 = a.views[v].tile_base, t1 = v + 1 < nv ? a.views[v + 1].tile_base : a.n_tiles;
        const int64_t b0 = a.views[v].depth_base, b1 = v + 1 < nv ? a.views[v + 1].depth_base : a.n_depth;
        const int64_t first = (wave % share) * 64 + lane, step = share * 64;
        for (int64_t t = t0 + first; t < t1; t += step) {
            float2 p[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) p[c] = *reinterpret_cast<const float2 *>(a.partial + 2 * (c * a.n_tiles + t));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                sS += p[c].x;
                sL += p[c].y;
            }
        }
        if (a.has_depth)
            for (int64_t b = b0 + first; b < b1; b += step) sD += a.depth_partial[b];
    }
    sS = wave_sum_f64(sS);
    sL = wave_sum_f64(sL);
    sD = wave_sum_f64(sD);
    if (lane == 0) {
        red[0][wave] = sS;
        red[1][wave] = sL;
        red[2][wave] = sD;
    }
    __syncthreads();
    const int u = v0 + (int)threadIdx.x;
    if ((int)threadIdx.x < at_once && u < nv) {
        const double npx = (double)a.views[u].W * (double)a.views[u].H;
        sS = sL = sD = 0.0;
        for (int i = 0; i < share; ++i) {
            sS += red[0][threadIdx.x * share + i];
            sL += red[1][threadIdx.x * share + i];
            sD += red[2][threadIdx.x * share + i];
        }
        const double l1 = sL / (3.0 * npx), dssim = sS / (3.0 * npx), ld = a.has_depth ? sD / npx : 0.0;
        const double lv = (1.0 - a.lam) * l1 + a.lam * dssim + (a.has_depth ? a.w_depth * ld : 0.0);
        out[threadIdx.x] = lv;
        a.loss[4 * u] = (float)l1;
        a.loss[4 * u + 1] = (float)(1.0 - dssim);
        a.loss[4 * u + 2] = (float)ld;
        a.loss[4 * u + 3] = (float)lv;
    }
}

// Calls of more views than one block takes at once: their terms, four views a block.
constexpr int kTermViews = 4;
__global__ __launch_bounds__(1024) void k_loss_views(FinalArgs a) {
    const int v0 = (int)blockIdx.x * kTermViews;
    view_terms(a, v0, kTermViews, 16 / kTermViews, a.terms + v0);
}

// One block of 16 waves: the terms of up to kArgViews views (of more, k_loss_views
// has left them), L_iso, and the total in view order.  The total is one chain of
// additions, so the terms are brought to LDS first.  With all views in rounds of
// 16 in this block and the chain over memory, 1024 views of 64 x 48 took 273 us here
// (the call 444 us; now 216, and 249 with two kernels before this one-pass loss).
__global__ __launch_bounds__(1024) void k_loss_final(FinalArgs a) {
    constexpr int kChunk = 1024;
    __shared__ double terms[kChunk], red[16];
    const int nv = a.views.n;
    double si = 0.0;
    for (int64_t b = threadIdx.x; b < a.n_iso_blocks; b += 1024) si += a.iso_partial[b];
    si = wave_sum_f64(si);
    if (lane_id() == 0) red[threadIdx.x >> 6] = si;
    if (nv <= kArgViews) view_terms(a, 0, nv, 16 / nv, terms);
    double total = 0.0;
    for (int v0 = 0; v0 < nv; v0 += kChunk) {
        const int n = nv - v0 < kChunk ? nv - v0 : kChunk;
        __syncthreads();  // the chunk before is added up
        if (nv > kArgViews && (int)threadIdx.x < n) terms[threadIdx.x] = a.terms[v0 + threadIdx.x];
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll 8
            for (int v = 0; v < n; ++v) total += terms[v];
        }
    }
    if (threadIdx.x != 0) return;
    double iso = 0.0;
    for (int w = 0; w < 16; ++w) iso += red[w];
    iso = a.n_gauss > 0 ? (double)a.w_iso * iso / (3.0 * (double)a.n_gauss) : 0.0;
    total += iso;
    a.loss[4 * nv] = (float)iso;
    a.loss[4 * nv + 1] = (float)total;
}

}  // namespace
}  // namespace mgs

using namespace mgs;

namespace {

mgs_status loss_check(const int32_t *sizes, int32_t n_views, const float *rgb, const float *gt_rgb,
                      const float *depth, const float *gt_depth, const float *scales, int64_t n_gauss,
                      const mgs_loss_opts *opts, const float *loss, const float *dL_drgb, const float *dL_ddepth,
                      const float *dL_dscales) {
    if (!sizes || !opts || !rgb || !gt_rgb || !loss || !dL_drgb) return MGS_ERR_INVALID_ARG;
    if (n_views <= 0 || n_views > 4096 || n_gauss < 0) return MGS_ERR_INVALID_ARG;
    if ((depth == nullptr) != (gt_depth == nullptr) || (depth && !dL_ddepth)) return MGS_ERR_INVALID_ARG;
    if (scales && n_gauss > 0 && !dL_dscales) return MGS_ERR_INVALID_ARG;
    if (!std::isfinite(opts->lambda_ssim) || !std::isfinite(opts->w_depth) || !std::isfinite(opts->w_iso))
        return MGS_ERR_INVALID_ARG;
    if (n_gauss >= (int64_t(1) << 31)) return MGS_ERR_TOO_LARGE;
    for (int v = 0; v < n_views; ++v) {
        const int32_t W = sizes[2 * v], H = sizes[2 * v + 1];
        if (W < 1 || H < 1 || W > 16384 || H > 16384) return MGS_ERR_INVALID_ARG;
    }
    return MGS_OK;
}

// Row chunks of an SSIM tile.  A tile of nch chunks yields 8 nch - 24 rows (the
// first 24 warm the two filters up), so tall tiles do less work, but a call must
// also fill the chip and end evenly.  In units of one block's chunk on a CU that
// holds several (0.75 us): a chunk takes a block alone three, and the last blocks
// of a call two and a half beyond their CU's share.  Measured: 641 x 479, 24.5 us
// at 5 chunks, 22.4 at 6, 24.9 at 7, 33 at 13; 8 x 1200 x 680, 234 us at 8, 214 at
// 13, 190 at 18, 182 at 20, 185 at 32.
// room: host room for n_views entries.
int ssim_chunks(const int32_t *sizes, int32_t n_views, LossView *room) {
    // consecutive views of one height together, H with their strips: the views of a
    // call mostly agree in size
    int runs = 0;
    for (int v = 0; v < n_views; ++v) {
        const int32_t H = sizes[2 * v + 1];
        if (runs == 0 || room[runs - 1].H != H) {
            room[runs].H = H;
            room[runs++].strips = 0;
        }
        room[runs - 1].strips += (sizes[2 * v] + kSC - 1) / kSC;
    }
    int best = 4;
    double least = 0.0;
    // every choice costs the host 6 us for 4096 different heights: a few will do there
    for (int nch = 4; nch <= 40; nch += runs > 256 ? 4 : 1) {
        // ceil(H / rows), exact: half a row off a whole number, which is a hundred times
        // what the float quotient can be off
        const float rows = (float)(8 * nch - kWarm), per_row = 1.0f / rows, up = rows - 0.5f;
        int64_t blocks = 0;
        for (int r = 0; r < runs; ++r) blocks += (int64_t)room[r].strips * (int32_t)(((float)room[r].H + up) * per_row);
        const double cost = nch * std::max(3.0, 3.0 * (double)blocks / 256.0 + 2.5);
        if (nch == 4 || cost < least) {
            least = cost;
            best = nch;
        }
    }
    return best;
}

bool overlap(const float *a, int64_t na, const float *b, int64_t nb) {
    if (!a || !b) return false;
    const uintptr_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
    return p < q + 4 * (uintptr_t)nb && q < p + 4 * (uintptr_t)na;
}

// The loss after the argument checks.  views: host room for n_views entries.
// ws == nullptr with ws_bytes == 0 only sizes the call (*ws_required).
mgs_status loss_run(const int32_t *sizes, int32_t n_views, const float *rgb, const float *gt_rgb,
                    const float *depth, const float *gt_depth, const float *scales, int64_t n_gauss,
                    const mgs_loss_opts *opts, LossView *views, void *ws, size_t ws_bytes, size_t *ws_required,
                    float *loss, float *dL_drgb, float *dL_ddepth, float *dL_dscales, void *stream) {
    const int nch = ssim_chunks(sizes, n_views, views);
    int64_t tiles = 0, P = 0, squares = 0, n_depth = 0;
    for (int v = 0; v < n_views; ++v) {
        const int32_t W = sizes[2 * v], H = sizes[2 * v + 1];
        LossView &L = views[v];
        L.W = W;
        L.H = H;
        L.strips = (int32_t)ceil_div(W, kSC);
        L.pad = 0;
        L.tile_base = (int32_t)tiles;  // the counts are checked below
        L.pix_base = P;
        L.depth_base = (int32_t)n_depth;
        L.inv_n3 = (float)(1.0 / (3.0 * (double)W * (double)H));
        L.inv_n1 = (float)(1.0 / ((double)W * (double)H));
        tiles += L.strips * ceil_div(H, 8 * nch - kWarm);
        squares += ceil_div(W, 32) * ceil_div(H, 32);
        if (depth) n_depth += ceil_div((int64_t)W * H, kDepthPix);
        P += (int64_t)W * H;
    }
    if (squares >= (int64_t(1) << 31) - 8) return MGS_ERR_TOO_LARGE;
    const bool iso = scales != nullptr && n_gauss > 0;
    const int64_t n_iso = iso ? ceil_div(n_gauss, kIsoGauss) : 0;
    if (3 * tiles + n_depth + n_iso >= (int64_t(1) << 31) - 16) return MGS_ERR_TOO_LARGE;
    Bump b;
    const size_t off_views = b.take(sizeof(LossView) * (size_t)n_views);
    // The size that the interface states, 36 bytes per pixel and 48 per 32x32
    // square, is what callers plan for; the partial sums take a part of it.
    const size_t off_part = b.take(4 * (size_t)9 * (size_t)P);
    b.take(4 * (size_t)12 * (size_t)squares);
    const size_t off_iso = b.take(8 * (size_t)std::max<int64_t>(iso ? ceil_div(n_gauss, 256) : 0, 1));
    const size_t off_terms = b.take(8 * (size_t)(n_views + 1));
    *ws_required = b.size();
    if (ws_bytes < b.size() || !ws) return MGS_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    ViewTable vt{};
    vt.n = n_views;
    const size_t view_bytes = sizeof(LossView) * (size_t)n_views;
    static_assert(sizeof(LossView) % 4 == 0, "views are copied as words");
    if (n_views <= kArgViews) {
        memcpy(vt.own, views, view_bytes);
    } else {
        vt.table = at<LossView>(ws, off_views);
        if (view_bytes <= 4 * (size_t)kArgCopyWords) {
            ArgWords aw;
            memcpy(aw.w, views, view_bytes);
            aw.n = (int32_t)(view_bytes / 4);
            k_arg_copy<<<1, 256, 0, s>>>(aw, at<uint32_t>(ws, off_views));
            MGS_LAUNCHED();
        } else {
            MGS_HIP(hipMemcpyAsync(at<void>(ws, off_views), views, view_bytes, hipMemcpyHostToDevice, s));
        }
    }
    float *partial = at<float>(ws, off_part), *depth_partial = partial + 6 * tiles;
    // Outputs over the images, which k_loss reads while it writes: the colour
    // gradient is formed behind the partial sums (24 bytes a tile of at least one
    // pixel and 4 a depth block leave the 12 a pixel), L_iso has a launch of its own.
    const auto over_images = [&](const float *out, int64_t n) {
        return overlap(out, n, rgb, 3 * P) || overlap(out, n, gt_rgb, 3 * P) || overlap(out, n, depth, P) ||
               overlap(out, n, gt_depth, P);
    };
    const bool put = over_images(dL_drgb, 3 * P), iso_after = iso && over_images(dL_dscales, 3 * n_gauss);
    SsimArgs a;
    a.views = vt;
    a.n_tiles = tiles;
    a.nch = nch;
    a.rgb = rgb;
    a.gt = gt_rgb;
    a.partial = partial;
    a.d_rgb = put ? depth_partial + n_depth : dL_drgb;
    a.lam = opts->lambda_ssim;
    {
        double w[kLW], sum = 0.0;
        for (int o = 0; o < kLW; ++o) {
            const double d = (double)(o - kLR);
            w[o] = std::exp(-d * d / (2.0 * 1.5 * 1.5));
            sum += w[o];
        }
        for (int o = 0; o < kLW; ++o) a.w[o] = (float)(w[o] / sum);
    }
    double *iso_part = at<double>(ws, off_iso);
    RestArgs r;
    r.n_depth = n_depth;
    r.depth = depth;
    r.gtd = gt_depth;
    r.d_depth = dL_ddepth;
    r.depth_partial = depth_partial;
    r.w_depth = opts->w_depth;
    r.scales = scales;
    r.n = iso ? n_gauss : 0;
    r.w_iso = opts->w_iso;
    r.d_scales = dL_dscales;
    r.iso_partial = iso_part;
    k_loss<<<(unsigned)(8 * ceil_div(3 * tiles, 8) + n_depth + (iso_after ? 0 : n_iso)), 256, 0, s>>>(a, r);
    MGS_LAUNCHED();
    if (put) {
        k_loss_put<<<(unsigned)std::min<int64_t>(ceil_div(3 * P, 1024), 4096), 256, 0, s>>>(a.d_rgb, dL_drgb, 3 * P);
        MGS_LAUNCHED();
    }
    if (iso_after) {
        a.n_tiles = r.n_depth = 0;
        k_loss<<<(unsigned)n_iso, 256, 0, s>>>(a, r);
        MGS_LAUNCHED();
    }
    FinalArgs f;
    f.views = vt;
    f.n_tiles = tiles;
    f.n_depth = n_depth;
    f.partial = partial;
    f.depth_partial = depth_partial;
    f.iso_partial = iso_part;
    f.n_iso_blocks = n_iso;
    f.n_gauss = iso ? n_gauss : 0;
    f.lam = opts->lambda_ssim;
    f.w_depth = opts->w_depth;
    f.w_iso = opts->w_iso;
    f.has_depth = depth != nullptr;
    f.terms = at<double>(ws, off_terms);
    f.loss = loss;
    if (n_views > kArgViews) {
        k_loss_views<<<(unsigned)ceil_div(n_views, kTermViews), 1024, 0, s>>>(f);
        MGS_LAUNCHED();
    }
    k_loss_final<<<1, 1024, 0, s>>>(f);
    MGS_LAUNCHED();
    return MGS_OK;
}

}  // namespace

extern "C" mgs_status mgs_mapping_loss(const int32_t *sizes, int32_t n_views, const float *rgb, const float *gt_rgb,
                                       const float *depth, const float *gt_depth, const float *scales,
                                       int64_t n_gauss, const mgs_loss_opts *opts, void *ws, size_t ws_bytes,
                                       size_t *ws_required, float *loss, float *dL_drgb, float *dL_ddepth,
                                       float *dL_dscales, void *stream) {
    ApiRange api_range("mgs_mapping_loss");
    if (!ws_required) return MGS_ERR_INVALID_ARG;
    const mgs_status st = loss_check(sizes, n_views, rgb, gt_rgb, depth, gt_depth, scales, n_gauss, opts, loss,
                                     dL_drgb, dL_ddepth, dL_dscales);
    if (st != MGS_OK) return st;
    std::vector<LossView> views((size_t)n_views);
    return loss_run(sizes, n_views, rgb, gt_rgb, depth, gt_depth, scales, n_gauss, opts, views.data(), ws,
                    ws_bytes, ws_required, loss, dL_drgb, dL_ddepth, dL_dscales, stream);
}

// ------------------------------------------------------- allocation-free entry
// The scratch of mgs_mapping_loss_noalloc: a fixed device array, one copy per
// GPU, held from the module's load until the process ends.  Host code never
// passes its name to a kernel (on the host it is only a stand-in for the
// symbol); it uses the device address that hipGetSymbolAddress returns for the
// current device, looked up once per device on the entry point's first call
// there.  Every call on one GPU shares the array: calls that overlap on one GPU
// (on different streams or host threads without ordering) race.  Nothing in it
// needs to start at zero: every kernel of the loss writes the scratch it later
// reads in the same call.
static __device__ __align__(256) unsigned char scratch[MGS_LOSS_SCRATCH_BYTES];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
std::atomic<void *> g_scratch_ptr[kScratchDevices];

// Device address of `scratch` on device `dev` (the current device).
mgs_status scratch_on(int dev, void **ptr) {
    if (dev < 0 || dev >= kScratchDevices) return MGS_ERR_INVALID_ARG;
    void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
        if (!p) {
            MGS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            if (!p) return MGS_ERR_HIP;
            g_scratch_ptr[dev].store(p, std::memory_order_release);
        }
    }
    *ptr = p;
    return MGS_OK;
}
}  // namespace

extern "C" mgs_status mgs_mapping_loss_noalloc(const int32_t *sizes, int32_t n_views, const float *rgb,
                                               const float *gt_rgb, const float *depth, const float *gt_depth,
                                               const float *scales, int64_t n_gauss, const mgs_loss_opts *opts,
                                               size_t *scratch_required, float *loss, float *dL_drgb,
                                               float *dL_ddepth, float *dL_dscales, void *stream) {
    ApiRange api_range("mgs_mapping_loss_noalloc");
    const mgs_status st = loss_check(sizes, n_views, rgb, gt_rgb, depth, gt_depth, scales, n_gauss, opts, loss,
                                     dL_drgb, dL_ddepth, dL_dscales);
    if (st != MGS_OK) return st;
    if (n_views > MGS_LOSS_NOALLOC_MAX_VIEWS) return MGS_ERR_SCRATCH;
    // few enough views for the view table to travel in kernel arguments: no
    // host-to-device copy
    static_assert(sizeof(LossView) * MGS_LOSS_NOALLOC_MAX_VIEWS <= 4 * (size_t)kArgCopyWords, "view table");
    LossView views[MGS_LOSS_NOALLOC_MAX_VIEWS];
    // size the call first: nothing is launched when it does not fit
    size_t need = 0;
    mgs_status r = loss_run(sizes, n_views, rgb, gt_rgb, depth, gt_depth, scales, n_gauss, opts, views, nullptr, 0,
                            &need, loss, dL_drgb, dL_ddepth, dL_dscales, stream);
    if (r != MGS_ERR_WORKSPACE) return r == MGS_OK ? MGS_ERR_HIP : r;
    if (scratch_required) *scratch_required = need;
    if (need > (size_t)MGS_LOSS_SCRATCH_BYTES) return MGS_ERR_SCRATCH;
    int dev = -1;
    MGS_HIP(hipGetDevice(&dev));
    if (stream) {
        int sdev = -1;
        MGS_HIP(hipStreamGetDevice(static_cast<hipStream_t>(stream), &sdev));
        if (sdev != dev) return MGS_ERR_INVALID_ARG;
    }
    void *ws = nullptr;
    r = scratch_on(dev, &ws);
    if (r != MGS_OK) return r;
    return loss_run(sizes, n_views, rgb, gt_rgb, depth, gt_depth, scales, n_gauss, opts, views, ws,
                    (size_t)MGS_LOSS_SCRATCH_BYTES, &need, loss, dL_drgb, dL_ddepth, dL_dscales, stream);
}
