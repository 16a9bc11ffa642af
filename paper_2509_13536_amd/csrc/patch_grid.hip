// Patch-Grid sampling of MemGS (Sec. II-B) for gfx950: new Gaussians from a
// keyframe's keypoints and from uniform samples in the patches where
// keypoints are sparse.
//
//   k_pg_count_one, or k_pg_fill and
//   k_pg_count    one thread per keypoint: its pixel (floor(u + 1/2)) and
//                 patch; integer atomics count the keypoints of each patch
//                 (exact, so the counts do not depend on the order)
//   k_pg_depth, k_pg_depth4
//                 one wave per candidate or four (the keypoints, then the s x s lattice
//                 of every patch): whether it is kept, and its depth, its own,
//                 the depth map's or the nearest keypoint's by a brute-force
//                 scan split over the lanes (fp32 squared distances, ties to the
//                 lower index); k_pg_resolve without keypoints
//   k_pg_write    order-preserving compaction of the kept candidates (many: a
//                 scan in two or three launches), back-projection through the
//                 pose and the new Gaussians' attributes (colour from the image,
//                 isotropic scale from the depth and the sample spacing)
// The nearest-keypoint search costs (candidates needing it) x (keypoints)
// fp32 distance evaluations, 64 lanes per candidate; keyframes hold a few
// thousand keypoints.
#include <cmath>

#include "api_range.hpp"
#include "common.hpp"
#include "scan.hpp"

namespace mgs {
namespace {

constexpr float kShC0 = 0.28209479177387814f;

struct PgArgs {
    int W, H, P, s, PX, PY, min_kp;
    int64_t n_kp, n_cand;
    const float *kp;        // [n_kp][2]
    const float *kp_depth;  // [n_kp]
    const float *depth_map; // [H][W] or null
    const float *image;     // [3][H][W]
    uint32_t *counts;       // [PX * PY]
    float *cand_z;          // [n_cand]: depth, 0 when dropped
};

// pixel of a keypoint, and whether it lies on the image
__device__ __forceinline__ bool kp_pixel(const PgArgs &a, int64_t i, int &x, int &y) {
    const float fx = floorf(a.kp[2 * i] + 0.5f), fy = floorf(a.kp[2 * i + 1] + 0.5f);
    if (!(fx >= 0.0f && fx < (float)a.W && fy >= 0.0f && fy < (float)a.H)) return false;  // NaN: false
    x = (int)fx;
    y = (int)fy;
    return true;
}

// pixel of lattice sample `lat` of patch `p` (over the patch's part of the image);
// candidates number below 2^31, so all divisions are of 32 bits
__device__ __forceinline__ void sample_pixel(const PgArgs &a, int p, int lat, int &x, int &y) {
    const int py = (int)((uint32_t)p / (uint32_t)a.PX), px = p - py * a.PX;
    const int l = lat / a.s, k = lat - l * a.s;
    const int w = min(a.P, a.W - a.P * px), h = min(a.P, a.H - a.P * py);
    x = a.P * px + ((2 * k + 1) * w) / (2 * a.s);
    y = a.P * py + ((2 * l + 1) * h) / (2 * a.s);
}

__global__ __launch_bounds__(256) void k_pg_fill(uint32_t *p, int64_t n, uint32_t *done) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
    if (i == 0) *done = 0u;
}

__global__ __launch_bounds__(256) void k_pg_count(PgArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n_kp) return;
    int x, y;
    if (kp_pixel(a, i, x, y)) atomicAdd(a.counts + (int64_t)(y / a.P) * a.PX + x / a.P, 1u);
}

// Both in one launch of one block, with the counts in LDS: 2000 keypoints over
// 836 patches are two a thread, and the launch saved is most of the cost.  A
// block alone takes about 1 us for each further 1024 keypoints, so up to eight.
constexpr int64_t kCountPatches = 8192, kCountKeypoints = 8192;
__global__ __launch_bounds__(1024) void k_pg_count_one(PgArgs a, int n_patch, uint32_t *done) {
    __shared__ uint32_t h[kCountPatches];
    for (int i = (int)threadIdx.x; i < n_patch; i += 1024) h[i] = 0u;
    if (threadIdx.x == 0) *done = 0u;
    __syncthreads();
    for (int i = (int)threadIdx.x; i < (int)a.n_kp; i += 1024) {
        int x, y;
        if (kp_pixel(a, i, x, y)) atomicAdd(&h[(y / a.P) * a.PX + x / a.P], 1u);
    }
    __syncthreads();
    for (int i = (int)threadIdx.x; i < n_patch; i += 1024) a.counts[i] = h[i];
}

// candidate depth still to be found by the nearest-keypoint search
constexpr float kNeedSearch = -1.0f;

// Candidate c's depth as far as it has its own or the depth map's (0: dropped,
// kNeedSearch: the nearest keypoint's), and its image position.
__device__ __forceinline__ float pg_own_depth(const PgArgs &a, int64_t c, float &qx, float &qy) {
    bool keep = false;
    float z = 0.0f;
    int x = 0, y = 0;
    if (c < a.n_kp) {
        keep = kp_pixel(a, c, x, y);
        qx = a.kp[2 * c];
        qy = a.kp[2 * c + 1];
        if (keep) {
            const float own = a.kp_depth[c];
            z = own > 0.0f ? own : 0.0f;
        }
    } else {
        const int j = (int)(c - a.n_kp), ss = a.s * a.s;
        const int p = (int)((uint32_t)j / (uint32_t)ss);
        keep = a.counts[p] < (uint32_t)a.min_kp;
        if (keep) sample_pixel(a, p, j - p * ss, x, y);
        qx = (float)x;
        qy = (float)y;
    }
    if (keep && z <= 0.0f && a.depth_map) {
        const float dm = a.depth_map[(int64_t)y * a.W + x];
        z = dm > 0.0f ? dm : 0.0f;
    }
    return !keep ? 0.0f : (z > 0.0f ? z : kNeedSearch);
}

// Without keypoints there is nothing to search: one thread per candidate.
__global__ __launch_bounds__(256) void k_pg_resolve(PgArgs a) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.n_cand) return;
    float qx, qy;
    const float z = pg_own_depth(a, c, qx, qy);
    a.cand_z[c] = z == kNeedSearch ? 0.0f : z;
}

// The depth of the keypoint nearest to (qx, qy), 0 without one that has a depth.  The
// lanes split the keypoints (lane l takes l, l + 64, ..., four in flight), keep
// their nearest with depth (fp32 squared distance, the first of equal ones), and a
// lexicographic (distance, index) minimum over the wave gives the nearest, ties to
// the lower index.
__device__ __forceinline__ float pg_nearest_depth(const PgArgs &a, float qx, float qy) {
    float best = INFINITY;
    int arg = (int)a.n_kp;  // none (n_kp < 2^31)
    constexpr int kAhead = 4;
    for (int64_t i0 = lane_id(); i0 < a.n_kp; i0 += 64 * kAhead) {
        float d[kAhead], kx[kAhead], ky[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int64_t i = min(i0 + 64 * u, a.n_kp - 1);  // repeated, the last changes nothing
            d[u] = a.kp_depth[i];
            kx[u] = a.kp[2 * i];
            ky[u] = a.kp[2 * i + 1];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const float dx = qx - kx[u], dy = qy - ky[u];
            const float d2 = dx * dx + dy * dy;
            if (d[u] > 0.0f && d2 < best) {
                best = d2;
                arg = (int)min(i0 + 64 * u, a.n_kp - 1);
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const float ob = __shfl_xor(best, off, 64);
        const int oa = __shfl_xor(arg, off, 64);
        if (ob < best || (ob == best && oa < arg)) {
            best = ob;
            arg = oa;
        }
    }
    return arg < a.n_kp ? a.kp_depth[arg] : 0.0f;
}

// One wave per candidate.  Bound by its chain of loads: 12 us for 5344 candidates and
// 2000 keypoints, where the search and a launch before it for the rest took 14 + 2.7.
__global__ __launch_bounds__(256) void k_pg_depth(PgArgs a) {
    const int64_t c = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (c >= a.n_cand) return;
    float qx, qy;
    float z = pg_own_depth(a, c, qx, qy);
    if (z == kNeedSearch) z = pg_nearest_depth(a, qx, qy);  // wave-uniform
    if (lane_id() == 0) a.cand_z[c] = z;
}

// A wave takes four candidates, a lane each for what they have of their own, and
// searches for those still without a depth in turn.
// Few candidates take a wave each: what a wave does for one of its own depth then
// costs less than searches in turn.  From kDepthMany on, where most are samples, a
// wave takes four: the whole call with a wave for one / four / sixteen, us, 2000
// keypoints: 25k candidates with a depth map 66 / 65 / 67, without 94 / 98 / 105;
// 51k 76 / 71 / 73, 127 / 128 / 146; 204k 125 / 92 / 90, 326 / 327 / 340; 816k 307 /
// 172 / 139, 1117 / 1118 / 1130.  Keypoints in the majority search longer: 50k of
// them, of 52k candidates, 1296 / 1428 / 1729.
constexpr int64_t kDepthMany = 32768;
__global__ __launch_bounds__(256) void k_pg_depth4(PgArgs a) {
    const int lane = lane_id();
    const int64_t c = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 4 + lane;
    if (c - lane >= a.n_cand) return;
    float qx = 0.0f, qy = 0.0f, z = 0.0f;
    const bool mine = lane < 4 && c < a.n_cand;
    if (mine) z = pg_own_depth(a, c, qx, qy);
    for (uint64_t left = ballot(mine && z == kNeedSearch); left; left &= left - 1ull) {
        const int l = __ffsll((long long)left) - 1;
        const float found = pg_nearest_depth(a, readlane_f(qx, l), readlane_f(qy, l));
        if (lane == l) z = found;
    }
    if (mine) a.cand_z[c] = z;
}

struct LoadKept {
    const float *z;
    __device__ uint32_t operator()(int64_t i) const { return z[i] > 0.0f ? 1u : 0u; }
};

struct PgWrite {
    PgArgs a;
    float R[9], t[3];
    float fx, fy, cx, cy;
    float opacity, scale_mul;  // scale = scale_mul * depth, scale_mul = factor * (P / s) / fx
    mgs_gaussians_out out;
    int32_t *source;
    __device__ void operator()(int64_t c, uint32_t o, uint32_t kept) const {
        if (!kept) return;
        int x, y;
        float qx, qy;
        if (c < a.n_kp) {
            kp_pixel(a, c, x, y);
            qx = a.kp[2 * c];
            qy = a.kp[2 * c + 1];
        } else {
            const int j = (int)(c - a.n_kp), ss = a.s * a.s;
            const int p = (int)((uint32_t)j / (uint32_t)ss);
            sample_pixel(a, p, j - p * ss, x, y);
            qx = (float)x;
            qy = (float)y;
        }
        const float z = a.cand_z[c];
        const float pc[3] = {z * (qx - cx) / fx - t[0], z * (qy - cy) / fy - t[1], z - t[2]};
        for (int k = 0; k < 3; ++k) out.means[3 * o + k] = R[k] * pc[0] + R[3 + k] * pc[1] + R[6 + k] * pc[2];
        const float sig = scale_mul * z;
        for (int k = 0; k < 3; ++k) out.scales[3 * o + k] = sig;
        out.quats[4 * o] = 1.0f;
        out.quats[4 * o + 1] = out.quats[4 * o + 2] = out.quats[4 * o + 3] = 0.0f;
        out.opac[o] = opacity;
        const int64_t plane = (int64_t)a.W * a.H, pix = (int64_t)y * a.W + x;
        for (int k = 0; k < 3; ++k) out.sh[3 * o + k] = (a.image[k * plane + pix] - 0.5f) / kShC0;
        if (source) source[o] = (int32_t)c;
    }
};

// Few candidates, in one launch: a block writes the kept ones of 256 candidates
// after counting those before them itself, and the block that ends last tells the
// host.  In place of block sums, scan and mail (3.9 + 15.8 + 3.6 us for 5344
// candidates, the scan's 2048 a block on three CUs) it takes 9.7.  A block reads up to
// kWriteDirect depths from L2, 64 a thread.
constexpr int64_t kWriteDirect = 16384;
__global__ __launch_bounds__(256) void k_pg_write(PgWrite w, uint32_t *total, uint32_t *done, uint32_t *mail,
                                                  uint32_t ticket) {
    __shared__ uint32_t lds[4];
    const int n = (int)w.a.n_cand, i = (int)blockIdx.x * 256 + (int)threadIdx.x;
    const LoadKept kept{w.a.cand_z};
    const uint32_t k = i < n ? kept(i) : 0u;
    uint32_t before = 0;
    for (int b = 0; b < (int)blockIdx.x; b += 8) {  // eight loads in flight
        uint32_t c[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) c[u] = b + u < (int)blockIdx.x ? kept((b + u) * 256 + (int)threadIdx.x) : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) before += c[u];
    }
    before = block_sum_u32(before, lds);
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan(k, lds, &tot);
    if (i < n) w(i, before + ex, k);
    const bool last = blockIdx.x == gridDim.x - 1;
    if (threadIdx.x == 0 && last) *total = before + tot;
    if (!mail) return;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(done, 1u) == gridDim.x - 1) mail_flag(mail, ticket);
}

}  // namespace
}  // namespace mgs

using namespace mgs;

extern "C" mgs_status mgs_patch_grid_sample(const mgs_camera *cam, const float *keypoints, const float *kp_depth,
                                            int64_t n_kp, const float *depth_map, const float *image,
                                            const mgs_pg_opts *opts, mgs_gaussians_out *out, int32_t *source,
                                            void *ws, size_t ws_bytes, size_t *ws_required, int64_t *n_out,
                                            void *stream) {
    ApiRange api_range("mgs_patch_grid_sample");
    if (!cam || !opts || !out || !ws_required || !n_out || !image) return MGS_ERR_INVALID_ARG;
    if (cam->width < 1 || cam->height < 1 || cam->width > 16384 || cam->height > 16384) return MGS_ERR_INVALID_ARG;
    if (!(cam->fx > 0.0f) || !(cam->fy > 0.0f) || !std::isfinite(cam->cx) || !std::isfinite(cam->cy))
        return MGS_ERR_INVALID_ARG;
    if (opts->patch < 1 || opts->samples < 1 || opts->samples > 64 || opts->min_keypoints < 0)
        return MGS_ERR_INVALID_ARG;
    if (!std::isfinite(opts->opacity) || !std::isfinite(opts->scale_factor)) return MGS_ERR_INVALID_ARG;
    if (n_kp < 0 || (n_kp > 0 && (!keypoints || !kp_depth))) return MGS_ERR_INVALID_ARG;
    if (!out->means || !out->scales || !out->quats || !out->opac || !out->sh) return MGS_ERR_INVALID_ARG;
    PgArgs a;
    a.W = cam->width;
    a.H = cam->height;
    a.P = opts->patch;
    a.s = opts->samples;
    a.PX = (int)ceil_div(a.W, a.P);
    a.PY = (int)ceil_div(a.H, a.P);
    a.min_kp = opts->min_keypoints;
    a.n_kp = n_kp;
    const int64_t n_patch = (int64_t)a.PX * a.PY;
    a.n_cand = n_kp + n_patch * a.s * a.s;
    if (a.n_cand >= (int64_t(1) << 31)) return MGS_ERR_TOO_LARGE;
    Bump b;
    const size_t off_counts = b.take(4 * (size_t)n_patch);
    const size_t off_z = b.take(4 * (size_t)a.n_cand);
    const size_t off_tmp = b.take(4 * (size_t)scan_tmp_words(a.n_cand));
    const size_t off_total = b.take(8);  // the kept count, and the blocks that have ended
    *ws_required = b.size();
    *n_out = 0;
    if (ws_bytes < b.size() || !ws) return MGS_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    a.kp = keypoints;
    a.kp_depth = kp_depth;
    a.depth_map = depth_map;
    a.image = image;
    a.counts = at<uint32_t>(ws, off_counts);
    a.cand_z = at<float>(ws, off_z);
    uint32_t *done = at<uint32_t>(ws, off_total) + 1;
    if (n_kp > 0 && n_kp <= kCountKeypoints && n_patch <= kCountPatches) {
        k_pg_count_one<<<1, 1024, 0, s>>>(a, (int)n_patch, done);
    } else {
        k_pg_fill<<<(unsigned)ceil_div(n_patch, 256), 256, 0, s>>>(a.counts, n_patch, done);
        if (n_kp > 0) k_pg_count<<<(unsigned)ceil_div(n_kp, 256), 256, 0, s>>>(a);
    }
    if (n_kp > 0 && a.n_cand >= kDepthMany && a.n_cand >= 4 * n_kp)
        k_pg_depth4<<<(unsigned)ceil_div(a.n_cand, 16), 256, 0, s>>>(a);
    else if (n_kp > 0)
        k_pg_depth<<<(unsigned)ceil_div(a.n_cand, 4), 256, 0, s>>>(a);
    else k_pg_resolve<<<(unsigned)ceil_div(a.n_cand, 256), 256, 0, s>>>(a);
    MGS_LAUNCHED();
    PgWrite w;
    w.a = a;
    for (int k = 0; k < 9; ++k) w.R[k] = cam->Tcw[4 * (k / 3) + k % 3];
    for (int k = 0; k < 3; ++k) w.t[k] = cam->Tcw[4 * k + 3];
    w.fx = cam->fx;
    w.fy = cam->fy;
    w.cx = cam->cx;
    w.cy = cam->cy;
    w.opacity = opts->opacity;
    w.scale_mul = (float)((double)opts->scale_factor * ((double)a.P / a.s) / (double)cam->fx);
    w.out = *out;
    w.source = source;
    // the kept count: to the host's mailbox word 9 when there is one
    const Mailbox mail = host_mailbox();
    uint32_t *total = mail.dev ? mail.dev + 9 : at<uint32_t>(ws, off_total);
    const uint32_t ticket = mail.host ? mailbox_ticket() : 0u;
    const bool direct = a.n_cand <= kWriteDirect;
    if (direct)
        k_pg_write<<<(unsigned)ceil_div(a.n_cand, 256), 256, 0, s>>>(w, total, done, mail.dev, ticket);
    else
        MGS_HIP(scan_exclusive(LoadKept{a.cand_z}, w, a.n_cand, at<uint32_t>(ws, off_tmp), total, s));
    MGS_LAUNCHED();
    uint32_t hn = 0;
    if (mail.host) {
        if (!direct) k_mail_done<<<1, 1, 0, s>>>(mail.dev, ticket);
        MGS_LAUNCHED();
        MGS_HIP(mailbox_wait(mail, ticket, s));
        hn = static_cast<const volatile uint32_t *>(mail.host)[9];
    } else {
        MGS_HIP(hipMemcpyAsync(&hn, total, 4, hipMemcpyDeviceToHost, s));
        MGS_HIP(hipStreamSynchronize(s));
    }
    *n_out = hn;
    return MGS_OK;
}
