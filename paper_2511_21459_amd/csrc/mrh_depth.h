// RGB-D fusion work units (Sec. 3.1 "Cameras", Eq. 2; Eq. 3 and Eq. 5; Sec. 3.2.1 merging
// criterion), shared by the single-map kernels (depth.hip) and the batched kernels (batch.hip).
//
//   depth_alloc_tile   a 16 x 16 pixel tile (one workgroup, each wave a 16 x 4 strip): back-
//                      projection, band walk over the block lattice, wave-deduplicated insert; new
//                      blocks are queued for the update
//   depth_cull         one thread per block that existed at the frame's start: conservative frustum
//                      test, visible blocks queued per level
//   depth_update_task  one queued level-0 or level-1 block (a wave), or 8 level-2 / 64 level-3
//                      blocks per wave: per-voxel projection and update, block variance bookkeeping
//                      and the merge of a block whose mean variance fell below the threshold
#pragma once

#include "mrh_update.h"

namespace mrh {

struct DepthFrame {
    int32_t parity;  // the frame's parity (selects the double-buffered per-frame counts)
    Pose P;
    double fx, fy, cx, cy, ifx, ify;
    int32_t width, height;
    const float MRH_GLOBAL* depth;  // device z-depth image, row-major
    double pixel_lim;  // 1/2 less the fast projection's margin
    // conservative culling of whole blocks (camera frame): side-plane normals and a range bound
    double plane[4][3];
    double cull_range;
    // largest valid depth per 16 x 16 pixel tile (written by the allocation launch, -1 when the
    // tile holds no valid sample), tiles_x tiles per row
    float MRH_GLOBAL* tile_max;
    int32_t tiles_x, tiles_y;
};

// Host: frame sizes the kernels accept (pixel indices 32-bit, pixel coordinates exact in FP32).
bool depth_size_ok(int32_t width, int32_t height);

// Host: enqueue the allocation and update launches of one RGB-D frame (rgb_dev: of a map with colour, else
// null; not checked).
mrh_status integrate_depth_frame(mrh_map* map, const float* depth_dev, const uint8_t* rgb_dev, int32_t width,
                                 int32_t height, const double K[4], const double T_ws[16]);

// Host: fill a frame descriptor; false on a non-finite pose or intrinsics or a zero focal length.
bool make_depth_frame(const mrh_config& cfg, const float* depth, int32_t width, int32_t height, const double K[4],
                      const double T_ws[16], DepthFrame& f);

// Nearest pixel of the voxel centre x (camera frame) under the projection of Eq. 2: the FP64
// evaluation u = fx (x0 (1 / x2)) + cx, pixel floor(u + 1/2), and likewise for v.  Returns the
// row-major pixel index, or -1 when x is not in front of the camera or falls outside the image.
__device__ inline int pixel_exact(const DepthFrame& f, double x0, double x1, double x2) {
    if (!(x2 > 0.0)) return -1;
    const double iz = 1.0 / x2;
    const double uu = (f.fx * (x0 * iz)) + f.cx;
    const double vv = (f.fy * (x1 * iz)) + f.cy;
    const double fu = __builtin_floor(uu + 0.5), fv = __builtin_floor(vv + 0.5);
    if (!(fu >= 0.0 && fu <= (double)(f.width - 1) && fv >= 0.0 && fv <= (double)(f.height - 1))) return -1;
    return (int)fv * f.width + (int)fu;
}

// The same decision with the division replaced: the hardware's FP32 reciprocal and one Newton step in FP64
// (relative error below 2^-44; FP64 issues at the FP32 rate here), taken only when u and v lie farther from
// a pixel boundary than the error can reach.  Returns -2 when it cannot decide.  The products, sums and the
// rounding of uu + 1/2 in the exact form stay below 1e-13 (|u| + |cx|) together with it, under the margin
// 1e-12 (larger side + |cx| + |cy| + 16) for every pixel of the image; a voxel beyond it whose error is larger is
// beyond it either way.  An FP32 evaluation left a voxel in 250 undecided, two per block, each
// with the exact form's divisions for the whole wave, and took more instructions for its margins (640 x 480
// room frames: update 24.8 -> 23.3 us).  `lam` receives |x| / x2 in FP32 for the range form (of use where a
// pixel is returned).  Straight-line code, as
// observe_form and the update of a group: a launch issued three quarter million branches and as many mask
// operations for what they skipped (with the grid below 29.1 -> 26.7 us).
__device__ inline int pixel_fast(const DepthFrame& f, double x0, double x1, double x2, float& lam) {
    const float xf0 = (float)x0, xf1 = (float)x1, xf2 = (float)x2;
    const float izf = __builtin_amdgcn_rcpf(xf2);
    lam = __builtin_amdgcn_sqrtf((xf0 * xf0 + xf1 * xf1) + xf2 * xf2) * izf;
    const double r = (double)izf;
    const double iz = __builtin_fma(r, __builtin_fma(-x2, r, 1.0), r);
    const double u = __builtin_fma(f.fx, x0 * iz, f.cx), v = __builtin_fma(f.fy, x1 * iz, f.cy);
    const double ru = __builtin_rint(u), rv = __builtin_rint(v);  // (ties are within the margin)
    const bool sure = (xf2 > 1e-6f) & (__builtin_fabs(u - ru) < f.pixel_lim) & (__builtin_fabs(v - rv) < f.pixel_lim);
    // clamped to the image, so that the conversions are defined
    const float fu = (float)ru, fv = (float)rv;
    const float cu = __builtin_amdgcn_fmed3f(fu, 0.0f, (float)(f.width - 1)), cv = __builtin_amdgcn_fmed3f(fv, 0.0f, (float)(f.height - 1));
    const int p = (int)(__umul24((uint32_t)cv, (uint32_t)f.width) + (uint32_t)cu);  // (sides are below 2^24)
    const int in = ((cu == fu) & (cv == fv)) ? p : -1;
    return x2 > 0.0 ? (sure ? in : -2) : -1;
}

// Observation of Eq. 2 (gate at -tau, truncation at +tau) for the voxel centre x from the depth d
// of its pixel, in FP64: the canonical evaluation.  False when the voxel is not updated.
__device__ inline bool observe_exact(const DevMap& m, double x0, double x1, double x2, double d, float& obs) {
    if (!(__builtin_isfinite(d) && d > 0.0 && d <= m.max_depth)) return false;
    double raw;
    if (m.form == MRH_FORM_RANGE) {
        const double iz = 1.0 / x2;
        const double nx = __builtin_sqrt((x0 * x0 + x1 * x1) + x2 * x2);
        raw = nx * ((d * iz) - 1.0);
    } else {
        raw = d - x2;
    }
    if (raw < -m.tau) return false;
    obs = (float)(raw < m.tau ? raw : m.tau);
    return true;
}

// The same observation with the range form's scale |x| / x2 in FP32 (`lam` from pixel_fast).
// Returns 1 (update with obs), 0 (no update) or 2 (undecided: observe_exact must decide).  The
// validity test is the canonical one (max_depth_f is the largest float not above max_depth) and
// the z-difference form is evaluated exactly (obs is of use where 1 is returned); the range-form value carries about 8 ulps (squares,
// sums, square root, reciprocal), so its -tau gate is taken only outside a 1e-5 tau band.
template <bool RANGE>
__device__ inline int observe_form(const DevMap& m, double x2, float lam, float d, float& obs) {
    const bool valid = (d > 0.0f) & (d <= __builtin_fminf(m.max_depth_f, 3.402823466e38f));
    const double ddiff = (double)d - x2;
    if (!RANGE) {
        obs = (float)(ddiff < m.tau ? ddiff : m.tau);
        return (valid & !(ddiff < -m.tau)) ? 1 : 0;
    }
    const float raw = (float)ddiff * lam;
    obs = raw < m.tau_f ? raw : m.tau_f;
    const bool close = __builtin_fabsf(raw + m.tau_f) <= 1e-5f * m.tau_f + 1e-6f * __builtin_fabsf(raw);
    return valid ? (close ? 2 : (raw < -m.tau_f ? 0 : 1)) : 0;
}
__device__ inline int observe_fast(const DevMap& m, double x2, float lam, float d, float& obs) {
    return m.form == MRH_FORM_RANGE ? observe_form<true>(m, x2, lam, d, obs) : observe_form<false>(m, x2, lam, d, obs);
}

// One voxel: pixel decision, depth lookup, observation; p receives the pixel.
__device__ inline bool observe(const DevMap& m, const DepthFrame& f, double x0, double x1, double x2, float& obs, int& p) {
    float lam;
    p = pixel_fast(f, x0, x1, x2, lam);
    const bool exact = p == -2;
    if (exact) p = pixel_exact(f, x0, x1, x2);
    if (p < 0) return false;
    const float d = f.depth[p];
    if (!exact) {
        const int r = observe_fast(m, x2, lam, d, obs);
        if (r != 2) return r == 1;
    }
    return observe_exact(m, x0, x1, x2, (double)d, obs);
}

// Screen rectangle of block (bx, by, bz), for the test below: with every block corner in front of the
// camera, each voxel centre projects inside the rectangle spanned by the projected corners (padded by a
// pixel against rounding) and lies at least as deep as the shallowest corner.  Returned as (that depth
// rounded down, first tile column | row << 16, tile columns | tiles << 16, -): depth -inf where the test
// says nothing, +inf and no tiles where the rectangle misses the image.  Evaluated by the cull, a thread per
// block: by the update, where all lanes of the block's wave repeat it, it took a quarter of the launch's
// vector instructions and its chain was on every task's path (640 x 480 room frames: update 26.7 -> 24.8 us;
// the allocation launch stays at 15.0, its cull ends before its tiles).  The corners in flight four at a time and
// without the division, since a batch's few cull workgroups have little else to hide them behind: a step of one
// map at 320 x 240, k_batch_alloc 16.2 -> 13.9 us (10.7 without rectangles, the update then 27.7 for 25.0).
__device__ inline u32x4 screen_rect(const DevMap& m, const DepthFrame& f, int32_t bx, int32_t by, int32_t bz) {
    const u32x4 unknown{0xFF800000u, 0u, 1u, 0u};
    double zmin = 1e300;
    int u0 = INT32_MAX, u1 = INT32_MIN, v0 = INT32_MAX, v1 = INT32_MIN;
#pragma unroll 4
    for (int c = 0; c < 8; ++c) {
        const double w0 = ((double)bx + (double)(c & 1)) * m.B - f.P.t[0];
        const double w1 = ((double)by + (double)((c >> 1) & 1)) * m.B - f.P.t[1];
        const double w2 = ((double)bz + (double)(c >> 2)) * m.B - f.P.t[2];
        const double x0 = (f.P.R[0][0] * w0 + f.P.R[1][0] * w1) + f.P.R[2][0] * w2;
        const double x1 = (f.P.R[0][1] * w0 + f.P.R[1][1] * w1) + f.P.R[2][1] * w2;
        const double x2 = (f.P.R[0][2] * w0 + f.P.R[1][2] * w1) + f.P.R[2][2] * w2;
        if (!(x2 > 1e-3)) return unknown;
        zmin = __builtin_fmin(zmin, x2);
        // (as in pixel_fast: off by 2^-44, against the pixel that the rectangle is padded by)
        const double r = (double)__builtin_amdgcn_rcpf((float)x2), iz = __builtin_fma(r, __builtin_fma(-x2, r, 1.0), r);
        const double u = __builtin_fmin(__builtin_fmax(f.fx * (x0 * iz) + f.cx, -1e8), 1e8);
        const double v = __builtin_fmin(__builtin_fmax(f.fy * (x1 * iz) + f.cy, -1e8), 1e8);
        u0 = min(u0, (int)__builtin_floor(u) - 1), u1 = max(u1, (int)__builtin_ceil(u) + 1);
        v0 = min(v0, (int)__builtin_floor(v) - 1), v1 = max(v1, (int)__builtin_ceil(v) + 1);
    }
    if (u1 < 0 || v1 < 0 || u0 > f.width - 1 || v0 > f.height - 1) return u32x4{0x7F800000u, 0u, 1u, 0u};
    const int tu0 = max(u0, 0) >> 4, tu1 = min(u1, f.width - 1) >> 4;
    const int tv0 = max(v0, 0) >> 4, tv1 = min(v1, f.height - 1) >> 4;
    const int ntu = tu1 - tu0 + 1;
    const int64_t nt = (int64_t)ntu * (tv1 - tv0 + 1);
    if (nt > 256 || tu0 > 0xFFFF || tv0 > 0xFFFF) return unknown;
    const float z = (float)(zmin * (1.0 - 1e-7));  // (not above zmin: the rounding is below 6e-8)
    return u32x4{__builtin_bit_cast(uint32_t, z), (uint32_t)tu0 | (uint32_t)tv0 << 16, (uint32_t)ntu | (uint32_t)nt << 16, 0u};
}

// Wave-uniform test of a block's screen rectangle (all lanes active): true when no voxel of the block can be
// updated by this frame.  If its depth exceeds every valid depth of the rectangle's tiles by more than tau,
// each voxel has x_z - d > tau for the depth d of its own pixel,
// so raw < -tau under both readings of Eq. 2 (the range reading scales x_z - d by |x| / x_z >= 1)
// and the gate rejects it; pixels outside the image or without a valid depth are never updated.
__device__ inline bool rect_hidden(const DevMap& m, const DepthFrame& f, const u32x4& r) {
    const int lane = lane_id(), ntu = (int)(r.z & 0xFFFFu), nt = (int)(r.z >> 16);
    const float MRH_GLOBAL* const first = f.tile_max + (size_t)(r.y >> 16) * f.tiles_x + (r.y & 0xFFFFu);
    const float inv = __builtin_amdgcn_rcpf((float)ntu);
    float dmax = -1.0f;
    for (int k = lane; k < nt; k += 64) {
        const int ty = (int)(((float)k + 0.5f) * inv);  // k / ntu (k < 256)
        dmax = __builtin_fmaxf(dmax, first[ty * f.tiles_x + (k - ty * ntu)]);
    }
    dmax = wave_max(dmax);
    const uint32_t zb = r.x;
    return (double)__builtin_bit_cast(float, zb) > (double)dmax + m.tau * (1.0 + 1e-6) + 1e-9;
}

__device__ inline bool block_visible(const DevMap& m, const DepthFrame& f, int64_t bx, int64_t by, int64_t bz) {
    const double hb = 0.5 * m.B;
    const double c[3] = {(double)bx * m.B + hb, (double)by * m.B + hb, (double)bz * m.B + hb};
    const double d0 = c[0] - f.P.t[0], d1 = c[1] - f.P.t[1], d2 = c[2] - f.P.t[2];
    double x[3];
    for (int r = 0; r < 3; ++r) x[r] = (f.P.R[0][r] * d0 + f.P.R[1][r] * d1) + f.P.R[2][r] * d2;
    const double rb = m.B * 0.8660254037844387 * (1.0 + 1e-9) + 1e-9;
    if (x[2] < -rb) return false;
    if (__builtin_sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]) - rb > f.cull_range) return false;
    for (int p = 0; p < 4; ++p)
        if (f.plane[p][0] * x[0] + f.plane[p][1] * x[1] + f.plane[p][2] * x[2] < -rb) return false;
    return true;
}

// Conservative frustum cull of the blocks that existed when the frame started, one thread per
// block: workgroup g of ng covers ids g * 256 + threadIdx, stepping by ng * 256.
__device__ inline void depth_cull(const DevMap& m, const DepthFrame& f, uint32_t g, uint32_t ng) {
    const uint32_t n = m.ctr->n_prev[f.parity];
    for (uint32_t base = g * blockDim.x; base < n; base += ng * blockDim.x) {
        const uint32_t id = base + threadIdx.x;
        int level = -1;
        uint32_t info = 0;
        unsigned long long key = 0;
        u32x4 rect{0u, 0u, 1u, 0u};
        if (id < n) {
            info = m.binfo[id];
            if (!(info & kNoBlockBit)) {
                key = m.bkey[id];
                int32_t bx, by, bz;
                unpack_key(key, bx, by, bz);
                if ((info & kNewBit) || block_visible(m, f, bx, by, bz)) level = (int)((info >> kLevelShift) & 3u);
                if (level == 0 || level == 1) rect = screen_rect(m, f, bx, by, bz);
            }
        }
        queue_block_wg(m, level, id, info, key, rect, f.parity);
    }
}

constexpr int kTileNew = 512;  // new blocks a tile registers with one allocation atomic

// One 16 x 16 pixel tile per workgroup (tile index `tile`, tiles_x tiles per row).  The keys a
// wave inserts are collected in LDS and registered with one atomic on the allocation word per
// workgroup; a key that finds the list full is registered by its wave directly.
__device__ inline void depth_alloc_tile(const DevMap& m, const DepthFrame& f, uint32_t tile, uint32_t tiles_x) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const float MRH_GLOBAL* __restrict__ depth = f.depth;
    const int u = (int)(tile % tiles_x) * 16 + (lane & 15);
    const int v = (int)(tile / tiles_x) * 16 + wave * 4 + (lane >> 4);
    bool ok = u < f.width && v < f.height;
    double d = 0.0;
    if (ok) {
        d = (double)depth[(int64_t)v * f.width + u];
        ok = __builtin_isfinite(d) && d > 0.0 && d <= m.max_depth;
    }
    Walk w;
    bool in_range = false;
    if (ok) {
        // back-projection of the pixel centre and the truncation band along the sensor ray
        const double ps[3] = {(((double)u - f.cx) * f.ifx) * d, (((double)v - f.cy) * f.ify) * d, d};
        double pw[3], n[3];
        pose_apply(f.P, ps, pw);
        unit_direction(pw, f.P.t, n);
        const double a[3] = {pw[0] - m.tau * n[0], pw[1] - m.tau * n[1], pw[2] - m.tau * n[2]};
        const double e[3] = {pw[0] + m.tau * n[0], pw[1] + m.tau * n[1], pw[2] + m.tau * n[2]};
        in_range = segment_in_range(a, e, m.invB);
        if (in_range) w.init(a, e, m.invB);
    }
    __shared__ uint32_t cnt[3];
    __shared__ float tmx[4];
    __shared__ unsigned long long nkey[kTileNew];
    __shared__ uint32_t nslot[kTileNew];
    __shared__ uint32_t ncount;
    __shared__ unsigned long long nold;
    if (threadIdx.x == 0) cnt[0] = cnt[1] = cnt[2] = ncount = 0;
    const float wmax = wave_max(ok ? (float)d : -1.0f);
    if (lane == 0) tmx[wave] = wmax;
    __syncthreads();
    const unsigned long long vmask = __ballot(ok), dmask = __ballot(ok && !in_range);
    if (lane == 0) {
        atomicAdd(&cnt[0], (uint32_t)__popcll(vmask));
        atomicAdd(&cnt[1], (uint32_t)__popcll(dmask));
    }
    bool active = in_range;
    uint32_t ncand = 0;  // keys this wave's walks produce (wave-uniform)
    while (unsigned long long amask = __ballot(active)) {
        ncand += (uint32_t)__popcll(amask);
        const unsigned long long key = active ? pack_key(w.c0, w.c1, w.c2) : 0ull;
        uint32_t slot = 0;
        const bool is_new = claim_keys(m, active, key, &slot);
        const unsigned long long newmask = __ballot(is_new);
        bool spill = false;
        if (newmask) {
            const int first = __ffsll((long long)newmask) - 1;
            uint32_t at = 0;
            if (lane == first) at = atomicAdd(&ncount, (uint32_t)__popcll(newmask));
            at = (uint32_t)__shfl((int)at, first) + (uint32_t)rank_in_mask(newmask);
            if (is_new) {
                if (at < (uint32_t)kTileNew) {
                    nkey[at] = key;
                    nslot[at] = slot;
                } else {
                    spill = true;
                }
            }
            register_new(m, spill, key, slot);
        }
        if (active) active = w.next();
    }
    if (lane == 0 && ncand) atomicAdd(&cnt[2], ncand);
    __syncthreads();
    const uint32_t nnew = ncount < (uint32_t)kTileNew ? ncount : (uint32_t)kTileNew;
    if (threadIdx.x == 0 && nnew) nold = take_new_blocks(m, nnew);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nnew; i += blockDim.x)
        register_block(m, nkey[i], nslot[i], (uint32_t)nold + i, (uint32_t)(nold >> 32) + i);
    if (threadIdx.x == 0) {
        stat_add(m, S_VALID, cnt[0]);
        stat_add(m, S_DROPPED, cnt[1]);
        stat_add(m, S_CAND, cnt[2]);
        f.tile_max[tile] = __builtin_fmaxf(__builtin_fmaxf(tmx[0], tmx[1]), __builtin_fmaxf(tmx[2], tmx[3]));
    }
}


// Camera-frame centre of voxel (i, j, k) of block b at `level`, canonical FP64.
__device__ inline void voxel_camera(const DevMap& m, const DepthFrame& f, int64_t bx, int64_t by, int64_t bz, int level,
                                    int i, int j, int k, double& x0, double& x1, double& x2) {
    const double nu = m.nu[level];
    const double c0 = (double)bx * m.B + ((double)i + 0.5) * nu;
    const double c1 = (double)by * m.B + ((double)j + 0.5) * nu;
    const double c2 = (double)bz * m.B + ((double)k + 0.5) * nu;
    const double d0 = c0 - f.P.t[0], d1 = c1 - f.P.t[1], d2 = c2 - f.P.t[2];
    x0 = (f.P.R[0][0] * d0 + f.P.R[1][0] * d1) + f.P.R[2][0] * d2;
    x1 = (f.P.R[0][1] * d0 + f.P.R[1][1] * d1) + f.P.R[2][1] * d2;
    x2 = (f.P.R[0][2] * d0 + f.P.R[1][2] * d1) + f.P.R[2][2] * d2;
}

// The projective decisions of lane group (I, J, K) of level-0 block (bx, by, bz): the 2x2x2 voxels
// 2I + a, 2J + b, 2K + c at Morton positions q = a + 2 b + 4 c.  pix[q] receives the voxel's pixel
// (-1: none), obs[q] its observation, and the returned mask has bit q set when the frame updates the
// voxel.
__device__ inline uint32_t fine_decisions(const DevMap& m, const DepthFrame& f, int32_t bx, int32_t by, int32_t bz, int I,
                                          int J, int K, int pix[8], float obs[8]) {
    const double nu = m.nu[0];
    // camera-frame products of R^T (c - t), one per axis coordinate of this lane's group
    double px[2][3], py[2][3], pz[2][3];
    for (int s = 0; s < 2; ++s) {
        const double cx = (double)bx * m.B + ((double)(2 * I + s) + 0.5) * nu;
        const double cy = (double)by * m.B + ((double)(2 * J + s) + 0.5) * nu;
        const double cz = (double)bz * m.B + ((double)(2 * K + s) + 0.5) * nu;
        const double dx = cx - f.P.t[0], dy = cy - f.P.t[1], dz = cz - f.P.t[2];
        for (int r = 0; r < 3; ++r) {
            px[s][r] = f.P.R[0][r] * dx;
            py[s][r] = f.P.R[1][r] * dy;
            pz[s][r] = f.P.R[2][r] * dz;
        }
    }
    // pixels first (the exact form only where the fast one cannot decide), then all depth loads at once, then
    // the observations; x recomputed by voxel_camera equals these sums bit for bit (same products, same
    // order, no contraction)
    float lam[8];
    uint32_t exact = 0;
#pragma unroll
    for (int ab = 0; ab < 4; ++ab) {  // (a pair of voxels shares the sum of two of its axes)
        const int a = ab & 1, b = ab >> 1;
        const double s0 = px[a][0] + py[b][0], s1 = px[a][1] + py[b][1], s2 = px[a][2] + py[b][2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int q = ab + 4 * c;
            pix[q] = pixel_fast(f, s0 + pz[c][0], s1 + pz[c][1], s2 + pz[c][2], lam[q]);
            exact |= (pix[q] == -2 ? 1u : 0u) << q;
            asm volatile("" : "+v"(lam[q]));  // here, not where it is used: it holds one register, its operands four
        }
    }
    for (uint32_t amb = exact; amb;) {
        const int q = __builtin_ctz(amb);
        amb &= amb - 1;
        double x0, x1, x2;
        voxel_camera(m, f, bx, by, bz, 0, 2 * I + (q & 1), 2 * J + ((q >> 1) & 1), 2 * K + (q >> 2), x0, x1, x2);
        const int p = pixel_exact(f, x0, x1, x2);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k == q) pix[k] = p;
    }
    float dq[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) dq[q] = f.depth[max(pix[q], 0)];
#pragma unroll
    for (int q = 0; q < 8; ++q) dq[q] = pix[q] >= 0 ? dq[q] : -1.f;
    uint32_t upd = 0, slow = 0;
    auto decide = [&](auto range) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double x2 = (px[q & 1][2] + py[(q >> 1) & 1][2]) + pz[q >> 2][2];
            const int fast = observe_form<decltype(range)::value>(m, x2, lam[q], dq[q], obs[q]);
            const int r = (exact >> q) & 1 ? (dq[q] > 0.f ? 2 : 0) : fast;
            upd |= r == 1 ? 1u << q : 0u;
            slow |= r == 2 ? 1u << q : 0u;
        }
    };
    if (m.form == MRH_FORM_RANGE) decide(std::true_type{});
    else decide(std::false_type{});
    // voxels the FP32 evaluation left undecided: the canonical evaluation from the same depth sample
    while (slow) {
        const int q = __builtin_ctz(slow);
        slow &= slow - 1;
        double x0, x1, x2;
        voxel_camera(m, f, bx, by, bz, 0, 2 * I + (q & 1), 2 * J + ((q >> 1) & 1), 2 * K + (q >> 2), x0, x1, x2);
        float o = 0.f, dsel = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k == q) dsel = dq[k];
        if (observe_exact(m, x0, x1, x2, (double)dsel, o)) {
            upd |= 1u << q;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k == q) obs[k] = o;
        }
    }
    return upd;
}

// A voxel's colour after the frame (Eq. 3 with w = 1, W the weight after it).
__device__ inline void color_update(const uint8_t* __restrict__ rgb, int p, uint32_t W, float c[3]) {
    const float inv = 1.0f / (float)W;
    for (int ch = 0; ch < 3; ++ch) c[ch] = c[ch] + ((float)rgb[3 * (size_t)p + ch] - c[ch]) * inv;
}

// Colours of a block that merged one level coarser, pooled as the TSDF was: the mean of the 8 children
// (the 8 lanes of a group) weighted by their weights Wp after the frame, into voxel `at` of C.
__device__ inline void pool_color8(float MRH_GLOBAL* C, size_t at, bool merged, uint32_t Wp, const float c[3]) {
    float sw = (float)Wp, s0 = sw * c[0], s1 = sw * c[1], s2 = sw * c[2];
    sw = group8_sum(sw);
    s0 = group8_sum(s0);
    s1 = group8_sum(s1);
    s2 = group8_sum(s2);
    if (!merged || (lane_id() & 7) != 0) return;
    const float inv = sw > 0.f ? 1.0f / sw : 0.f;
    C[3 * at] = s0 * inv;
    C[3 * at + 1] = s1 * inv;
    C[3 * at + 2] = s2 * inv;
}

// The same for a level-0 block's lane group (Morton positions 8l .. 8l+7), whose colours are stored, or pooled
// into voxel l of level-1 slot `now` when the block merged: upd and pix as fine_decisions returned them,
// W the weights after the frame as stored, Wp before they were rounded.
__device__ inline void color_fine_group(const DevMap& m, const uint8_t* __restrict__ rgb, uint32_t info, uint32_t now, uint32_t upd,
                                        bool fresh, bool merged, const int pix[8], const uint32_t W[8], const uint32_t Wp[8]) {
    const int lane = lane_id();
    float c[24];
    float MRH_GLOBAL* cp = m.C[0] + 3 * ((size_t)(info & kSlotMask) * 512 + (size_t)lane * 8);  // 96 B, 16 B aligned
    if (fresh || (!merged && !upd)) {
        for (int k = 0; k < 24; ++k) c[k] = 0.f;
    } else {
        for (int k = 0; k < 6; ++k) {
            const f32x4 v = load_as<f32x4>(cp + 4 * k);
            c[4 * k] = v.x, c[4 * k + 1] = v.y, c[4 * k + 2] = v.z, c[4 * k + 3] = v.w;
        }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if ((upd >> q) & 1) color_update(rgb, pix[q], merged ? Wp[q] : W[q], c + 3 * q);
    if (!merged) {
        if (upd || fresh)
            for (int k = 0; k < 6; ++k) store_as(cp + 4 * k, f32x4{c[4 * k], c[4 * k + 1], c[4 * k + 2], c[4 * k + 3]});
        return;
    }
    float sw = 0.f, s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float w = (float)Wp[q];
        sw += w;
        s0 += w * c[3 * q];
        s1 += w * c[3 * q + 1];
        s2 += w * c[3 * q + 2];
    }
    const float inv = sw > 0.f ? 1.0f / sw : 0.f;
    float MRH_GLOBAL* Cc = m.C[1] + 3 * ((size_t)(now & kSlotMask) * 64 + (size_t)lane);
    Cc[0] = s0 * inv;
    Cc[1] = s1 * inv;
    Cc[2] = s2 * inv;
}

// Level-0 block: lane l owns the 2x2x2 group of Morton positions 8l .. 8l+7.
template <int ST, bool COLOR>
__device__ inline TaskOut integrate_fine_block(const DevMap& m, const DepthFrame& f, const uint8_t* __restrict__ rgb,
                                               const u32x4 eq, const u32x4 rect) {
    const int lane = lane_id();
    const u32x4 e = uniform(eq);  // one block per wave
    const uint32_t id = e.x, info = e.y;
    if (info & kNoBlockBit) return TaskOut{};
    int32_t bx, by, bz;
    unpack_key(entry_key(e), bx, by, bz);
    const bool fresh = (info & kNewBit) != 0;
    const double bvs = m.bvsum[id];
    const uint32_t bvc = m.bvcnt[id];
    if (!fresh && rect_hidden(m, f, uniform(rect))) return TaskOut{};
    int I, J, K;
    demorton3(lane, I, J, K);
    int pix[8];
    float obs[8];
    const uint32_t upd = fine_decisions(m, f, bx, by, bz, I, J, K, pix, obs);
    const int nupd = wave_sum((int)__popc(upd));
    if (nupd == 0 && !fresh) return TaskOut{};
    TaskOut out;
    out.obs = (uint32_t)nupd;
    out.fresh = fresh ? (uint32_t)nupd : 0u;

    const size_t base = (size_t)(info & kSlotMask) * 512 + (size_t)lane * 8;
    float D[8], S2[8];
    uint32_t W[8];
    bool have = false;
    if (fresh) {
        for (int q = 0; q < 8; ++q) D[q] = 0.f, S2[q] = 0.f, W[q] = 0u;
        have = true;
    } else if (upd) {
        Store<ST>::get8(m, base, D, W, S2);
        have = true;
    }
    double dsum = 0.0;
    int dcnt = 0;
    uint32_t Wp[8];  // (colour) the weights after the frame, not rounded
    if (COLOR && have)
        for (int q = 0; q < 8; ++q) Wp[q] = W[q] + ((upd >> q) & 1);
    if (upd) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bool u = (upd >> q) & 1;
            float d = D[q], s2 = S2[q];
            uint32_t w = W[q];
            welford(obs[q], d, w, s2);
            Store<ST>::round(m, d, w, s2);
            const double change = var_term(m, w, s2) - var_term(m, W[q], S2[q]);
            dsum += u ? change : 0.0;
            dcnt += u ? var_count(m, w) - var_count(m, W[q]) : 0;
            D[q] = u ? d : D[q];
            S2[q] = u ? s2 : S2[q];
            W[q] = u ? w : W[q];
        }
    }
    out.merge0 = (uint32_t)finish_fine<ST>(m, id, info, D, W, S2, have, upd != 0 || fresh, nupd, dsum, dcnt,
                                                        bvs, bvc, f.parity);
    if (COLOR) {
        uint32_t now = 0;
        if (out.merge0) {
            DeferList::sync();
            now = uniform(m.binfo[id]);
            if (!have)  // (finish_fine read the group)
                for (int q = 0; q < 8; ++q) Wp[q] = W[q];
        }
        color_fine_group(m, rgb, info, now, upd, fresh, out.merge0 != 0, pix, W, Wp);
    }
    return out;
}

// Level-1 block: lane l owns the voxel at Morton position l.
template <int ST, bool COLOR>
__device__ inline TaskOut integrate_level1_block(const DevMap& m, const DepthFrame& f, const uint8_t* __restrict__ rgb,
                                                 const u32x4 eq, const u32x4 rect) {
    const int lane = lane_id();
    const u32x4 e = uniform(eq);  // one block per wave
    const uint32_t id = e.x, info = e.y;
    int32_t bx, by, bz;
    unpack_key(entry_key(e), bx, by, bz);
    const double bvs = m.bvsum[id];
    const uint32_t bvc = m.bvcnt[id];
    if (rect_hidden(m, f, uniform(rect))) return TaskOut{};
    int i, j, k;
    demorton3(lane, i, j, k);
    double x0, x1, x2;
    voxel_camera(m, f, bx, by, bz, 1, i, j, k, x0, x1, x2);
    float obs = 0.f;
    int pix;
    const bool upd = observe(m, f, x0, x1, x2, obs, pix);
    const int nupd = __popcll(__ballot(upd));
    if (nupd == 0) return TaskOut{};
    TaskOut out;
    out.obs = (uint32_t)nupd;
    const size_t at = (size_t)(info & kSlotMask) * 64 + lane;
    float D, S2;
    uint32_t W;
    Store<ST>::get(m, 1, at, D, W, S2);
    const uint32_t Wp = W + (upd ? 1u : 0u);
    double dsum = 0.0;
    int dcnt = 0;
    if (upd) {
        const double before = var_term(m, W, S2);
        const int cb = var_count(m, W);
        welford(obs, D, W, S2);
        Store<ST>::round(m, D, W, S2);
        dsum = var_term(m, W, S2) - before;
        dcnt = var_count(m, W) - cb;
    }
    out.merge1 = (uint32_t)finish_coarse<ST>(m, id, info, 1, D, W, S2, upd, nupd, dsum, dcnt, bvs, bvc,
                                                          f.parity);
    if (COLOR) {
        const bool merged = out.merge1 != 0;
        float c[3];
        for (int ch = 0; ch < 3; ++ch) c[ch] = m.C[1][3 * at + ch];
        if (upd) color_update(rgb, pix, merged ? Wp : W, c);
        if (merged) {
            DeferList::sync();
            pool_color8(m.C[2], (size_t)(m.binfo[id] & kSlotMask) * 8 + (size_t)(lane >> 3), true, Wp, c);
        } else if (upd) {
            for (int ch = 0; ch < 3; ++ch) m.C[1][3 * at + ch] = c[ch];
        }
    }
    return out;
}

// 64 / seg blocks of `level` (2: seg = 8 voxels, 3: seg = 1 voxel) per wave.
template <int ST, bool COLOR>
__device__ inline TaskOut integrate_packed_blocks(const DevMap& m, const DepthFrame& f, const uint8_t* __restrict__ rgb,
                                               const u32x4 MRH_GLOBAL* list, uint32_t count, uint32_t group, int level) {
    const int lane = lane_id();
    const int seg = level == 2 ? 8 : 1;
    const uint32_t bi = group * (uint32_t)(64 / seg) + (uint32_t)(lane / seg);
    const bool live = bi < count;
    uint32_t id = 0, info = 0;
    bool upd = false;
    float obs = 0.f;
    int pix = 0;
    if (live) {
        const u32x4 e = list[bi];
        id = e.x;
        info = e.y;
        int32_t bx, by, bz;
        unpack_key(entry_key(e), bx, by, bz);
        int i, j, k;
        demorton3(lane % seg, i, j, k);
        double x0, x1, x2;
        voxel_camera(m, f, bx, by, bz, level, i, j, k, x0, x1, x2);
        upd = observe(m, f, x0, x1, x2, obs, pix);
    }
    if (!__ballot(upd)) return TaskOut{};
    float D = 0.f, S2 = 0.f;
    uint32_t W = 0;
    double dsum = 0.0;
    int dcnt = 0;
    uint32_t Wp = 0;  // the weight after the frame, not rounded
    if (upd) {
        Store<ST>::get(m, level, (size_t)(info & kSlotMask) * seg + (lane % seg), D, W, S2);
        Wp = W + 1u;
        const double before = var_term(m, W, S2);
        const int cb = var_count(m, W);
        welford(obs, D, W, S2);
        Store<ST>::round(m, D, W, S2);
        dsum = var_term(m, W, S2) - before;
        dcnt = var_count(m, W) - cb;
    } else if (live && seg > 1) {
        // a segment whose block merges needs all of its voxels
        Store<ST>::get(m, level, (size_t)(info & kSlotMask) * seg + (lane % seg), D, W, S2);
        Wp = W;
    }
    TaskOut out;
    out.obs = (uint32_t)wave_sum(upd ? 1 : 0);
    const int merge = finish_packed<ST>(m, live, id, info, level, seg, D, W, S2, upd, upd ? 1 : 0, dsum, dcnt);
    out.merge2 = (uint32_t)wave_sum(merge);
    if (COLOR) {
        const bool merged = seg == 8 && group8_sum(merge) != 0;
        const size_t at = 3 * ((size_t)(info & kSlotMask) * seg + (lane % seg));
        float MRH_GLOBAL* const C = level == 2 ? m.C[2] : m.C[3];
        float c[3] = {0.f, 0.f, 0.f};
        if (upd || (merged && live))
            for (int ch = 0; ch < 3; ++ch) c[ch] = C[at + ch];
        if (upd) color_update(rgb, pix, merged ? Wp : W, c);
        if (upd && !merged)
            for (int ch = 0; ch < 3; ++ch) C[at + ch] = c[ch];
        if (seg == 8 && __ballot(merged)) {
            DeferList::sync();
            const uint32_t now = merged ? m.binfo[id] : 0u;
            pool_color8(m.C[3], (size_t)(now & kSlotMask), merged, Wp, c);
        }
    }
    return out;
}

// One update task t of the frame's task space (see TaskCounts).
template <int ST, bool COLOR>
__device__ inline TaskOut depth_update_task(const DevMap& m, const DepthFrame& f, const uint8_t* __restrict__ rgb, uint32_t t,
                                            const TaskCounts& c) {
    const uint32_t n0 = c.n[0] + c.n_new;
    const uint32_t g2 = (c.n[2] + 7) / 8;
    // each work unit is called in one place: its code is inlined there
    if (t < n0) {
        const uint32_t id = c.new_base + (t - c.n[0]);
        u32x4 e, rect{0u, 0u, 1u, 0u};
        if (t < c.n[0]) e = m.vis[0][t], rect = m.vrect[0][t];
        else e = make_entry(id, m.binfo[id], m.bkey[id]);  // (new: not tested)
        return integrate_fine_block<ST, COLOR>(m, f, rgb, e, rect);
    }
    if (t < n0 + c.n[1]) return integrate_level1_block<ST, COLOR>(m, f, rgb, m.vis[1][t - n0], m.vrect[1][t - n0]);
    const uint32_t g = t - n0 - c.n[1];
    const int level = g < g2 ? 2 : 3;
    return integrate_packed_blocks<ST, COLOR>(m, f, rgb, m.vis[level], c.n[level], level == 2 ? g : g - g2, level);
}

}  // namespace mrh
