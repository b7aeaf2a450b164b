// Multi-resolution trilinear SDF query (Sec. 3.4) and its adjoint for points and a 6-DoF pose.
//
// Four lanes per point, two corners each.  The point's block fixes the interpolation lattice (its level n); each of
// the 8 surrounding level-n lattice points takes the TSDF of the voxel, at whatever level its own
// block has, whose cell contains it; corners without a block or with W = 0 drop out and the
// remaining trilinear weights are renormalised.  Lattice indices and weights are FP64.
#include <cmath>

#include "mrh_store.h"

namespace mrh {

struct QueryParams {
    Pose P;
    int32_t identity;
    int32_t strict;
};

// The query of one point by 4 consecutive lanes: lane c = lane & 3 takes corners c and c + 4 (the two
// along z); every lane of the group calls with the same x.  A query is a chain of reads (its block's
// hash slot, the corners' slots, the voxels) behind about 1100 instructions when one lane does all 8
// corners, which leaves the chip idle on small batches.  Measured with gradients on a 1 cm room, one / 8 / 4 lanes
// per point: 1000 points 14 / 7 / 8 us, 65536 24 / 15 / 14 us, 1M in
// random order 151 / 119 / 121 us (bound by the lines met; 78 us once D and W share theirs), 1M in
// block order 74 / 93 / 60 us (bound by VALU issue, where the work that 8 lanes repeat shows).
struct QueryResult {
    bool valid;      // the same on the group's lanes, as are the values
    double sdf;
    double grad[3];  // d sdf / d x (world)
};

// Sum over each group of 4 consecutive lanes, on every lane.
__device__ inline double group4_sum(double v) {
    v += dpp<kDppXor1>(v);
    return v + dpp<kDppXor2>(v);
}

// The hash slot content of block (x, y, z).
__device__ inline HashSlot block_slot(const DevMap& m, int32_t x, int32_t y, int32_t z) {
    const unsigned long long key = pack_key(x, y, z);
    const uint32_t h = spatial_hash(x, y, z) & m.hmask;
    return follow_slot(m, key, h, load_slot(m, h));
}

// The row of the point's block, NOBLOCK where it has none.
__device__ inline uint32_t home_row(const DevMap& m, const double x[3]) {
    int32_t b[3];
    bool in_range = true;
    for (int k = 0; k < 3; ++k) {
        const double fb = __builtin_floor(x[k] * m.invB);
        in_range = in_range && __builtin_fabs(fb) <= (double)kKeyLimit;
        b[k] = (int32_t)fb;
    }
    return in_range ? block_slot(m, b[0], b[1], b[2]).info : kNoBlockBit;
}

template <int ST, bool GRAD>
__device__ inline QueryResult query_point(const DevMap& m, const double x[3], uint32_t info, bool strict) {
    QueryResult q;
    q.valid = false;
    q.sdf = 0.0;
    q.grad[0] = q.grad[1] = q.grad[2] = 0.0;
    const int c = lane_id() & 3;
    // uniform over the group, so its lanes leave together and the sums below see all 4
    if (info & kNoBlockBit) return q;
    int32_t b[3];
    for (int k = 0; k < 3; ++k) b[k] = (int32_t)__builtin_floor(x[k] * m.invB);
    const int n = (int)((info >> kLevelShift) & 3u), shift = 3 - n;
    // lattice cell, fractions, and this lane's corners: lattice points cell + (dx, dy, 0 and 1), each in
    // block cell >> shift (floor division by the block side)
    int32_t cell[3];
    double f[3];
    const double inv_nu = inv_nu_of(m.inv_nu, n);
    for (int k = 0; k < 3; ++k) {
        const double g = x[k] * inv_nu - 0.5;
        const double fl = __builtin_floor(g);
        f[k] = g - fl;
        cell[k] = (int32_t)fl;
    }
    const bool dx = (c & 1) != 0, dy = (c & 2) != 0;
    cell[0] += dx ? 1 : 0;
    cell[1] += dy ? 1 : 0;
    const int32_t bx = cell[0] >> shift, by = cell[1] >> shift, bz0 = cell[2] >> shift, bz1 = (cell[2] + 1) >> shift;
    const bool side = bx != b[0] || by != b[1];
    uint32_t row[2] = {info, info};
    {
        // both home slots are read before either is examined
        const bool need0 = side || bz0 != b[2], need1 = (side || bz1 != b[2]) && bz1 != bz0;
        const unsigned long long k0 = pack_key(bx, by, bz0), k1 = pack_key(bx, by, bz1);
        const uint32_t h0 = spatial_hash(bx, by, bz0) & m.hmask, h1 = spatial_hash(bx, by, bz1) & m.hmask;
        HashSlot s0{k0, 0u, info}, s1{k1, 0u, info};
        if (need0) s0 = load_slot(m, h0);
        if (need1) s1 = load_slot(m, h1);
        row[0] = follow_slot(m, k0, h0, s0).info;
        row[1] = follow_slot(m, k1, h1, s1).info;
        if (bz1 == bz0) row[1] = row[0];
    }
    double cd[2] = {0.0, 0.0};
    bool have[2] = {false, false};
    {
        const int base[2] = {bz0, bz1};
        uint32_t W[2] = {0u, 0u};
        float D[2] = {0.f, 0.f};
        for (int z = 0; z < 2; ++z) {
            if (row[z] & kNoBlockBit) continue;
            const int n2 = (int)((row[z] >> kLevelShift) & 3u);
            // lattice point (cell + 1/2) nu_n in half finest-voxel units, relative to its block
            const int i = ((2 * (cell[0] - (bx << shift)) + 1) << n) >> (n2 + 1);
            const int j = ((2 * (cell[1] - (by << shift)) + 1) << n) >> (n2 + 1);
            const int k = ((2 * (cell[2] + z - (base[z] << shift)) + 1) << n) >> (n2 + 1);
            const size_t at = ((size_t)(row[z] & kSlotMask) << (3 * (3 - n2))) +
                              (size_t)(spread3(i) | (spread3(j) << 1) | (spread3(k) << 2));
            Store<ST>::getDW(m, n2, at, D[z], W[z]);
        }
        for (int z = 0; z < 2; ++z) {
            have[z] = W[z] != 0u;
            cd[z] = have[z] ? (double)D[z] : 0.0;
        }
    }
    const double wx = dx ? f[0] : 1.0 - f[0], wy = dy ? f[1] : 1.0 - f[1], wxy = wx * wy;
    const double cw[2] = {have[0] ? wxy * (1.0 - f[2]) : 0.0, have[1] ? wxy * f[2] : 0.0};
    const double wsum = group4_sum(cw[0] + cw[1]);
    const double num = group4_sum(cw[0] * cd[0] + cw[1] * cd[1]);
    // all 8 corners observed, or one observed with a positive weight, over the group's 4 bits
    const int sh = lane_id() & 60;
    const uint32_t seen = (uint32_t)(__ballot(have[0] && have[1]) >> sh) & 15u;
    const uint32_t pos = (uint32_t)(__ballot(cw[0] > 0.0 || cw[1] > 0.0) >> sh) & 15u;
    if (strict ? seen != 15u : pos == 0u) return q;
    q.valid = true;
    q.sdf = num / wsum;
    if (GRAD) {
        const double e0 = have[0] ? cd[0] - q.sdf : 0.0, e1 = have[1] ? cd[1] - q.sdf : 0.0;
        const double ez = (1.0 - f[2]) * e0 + f[2] * e1;
        const double r = inv_nu / wsum;
        q.grad[0] = group4_sum((dx ? wy : -wy) * ez) * r;
        q.grad[1] = group4_sum((dy ? wx : -wx) * ez) * r;
        q.grad[2] = group4_sum(wxy * (e1 - e0)) * r;
    }
    return q;
}

__device__ inline void world_point(const QueryParams& qp, const float* pts, int64_t i, double x[3]) {
    const double p[3] = {(double)pts[3 * i], (double)pts[3 * i + 1], (double)pts[3 * i + 2]};
    if (qp.identity) {
        x[0] = p[0], x[1] = p[1], x[2] = p[2];
    } else {
        pose_apply(qp.P, p, x);
    }
}

constexpr int kQueryPoints = 64;  // points per 256-thread workgroup

// Batches of at least kQueryMany points: a wave first looks up the blocks of 64 points, a lane each, and then goes
// on with those that have one, four lanes each (src, of the 64).  A batch that fills the chip is bound by VALU issue
// or by the lines met, and four lanes that repeat a lookup cost what they save in a small one.  1M / 4M points on a
// 1 cm room, us, one lane per point / four / this: off the map 17 / 23 / 16 and 48 / 72 / 41; over the map's box
// 59 / 39 / 30 and 193 / 132 / 91; random on the map 142 / 75 / 77 and 539 / 276 / 283; with the adjoint in block
// order 93 / 95 / 86 and 238 / 267 / 214, off the map 42 / 58 / 44 and 66 / 132 / 70.  32 points per wave: off the
// map 17 and 47, over its box 32 and 94.  Below kQueryMany forward queries gain nothing from the lookup apart (262144
// points: random on a street 33 us by it, 31 by four lanes; over a box 17 and 22; off the map 15 either way).  The
// adjoint, whose fewer workgroups loop, has it from kAdjointMany points on: 131072 off the map 36 us by one lane
// per point, 40 by four, 36 by it; over a street's box 46, 43 and 39; on the street 63, 50 and 55.
constexpr int64_t kQueryMany = 1 << 19, kAdjointMany = 1 << 17;
constexpr int kQueryWave = 64;

template <typename F>
__device__ inline void query_many(const DevMap& m, const QueryParams& qp, const float* __restrict__ pts, int64_t n, F&& point) {
    const int lane = lane_id();
    const int64_t stride = (int64_t)gridDim.x * 4 * kQueryWave;
    for (int64_t first = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kQueryWave; first < n; first += stride) {
        const bool on = first + lane < n;
        double x[3] = {0.0, 0.0, 0.0};
        uint32_t info = kNoBlockBit;
        if (on) {
            world_point(qp, pts, first + lane, x);
            info = home_row(m, x);
        }
        const unsigned long long present = __ballot(!(info & kNoBlockBit));
        if (on && (info & kNoBlockBit)) point(first + lane, x, kNoBlockBit, false);
        const int count = __popcll(present);
        for (int k = 0; k < count; k += kQueryWave / 4) {
            const int at = k + (lane >> 2);
            const int src = count == kQueryWave ? at : nth_bit(present, min(at, count - 1));
            double xs[3];
            for (int a = 0; a < 3; ++a) xs[a] = __shfl(x[a], src);
            const uint32_t is = (uint32_t)__shfl((int)info, src);
            if (at < count) point(first + src, xs, is, true);
        }
    }
}

template <int ST, bool GRAD>
__global__ __launch_bounds__(256, 8) void k_query_many(const DevMap* __restrict__ pm, QueryParams qp, const float* __restrict__ pts,
                                                       int64_t n, float* sdf, uint8_t* valid, float* grad) {
    const DevMap& m = *pm;
    const int c = lane_id() & 3;
    query_many(m, qp, pts, n, [&](int64_t i, const double x[3], uint32_t info, bool present) {
        if (!present) {
            sdf[i] = 0.f;
            valid[i] = 0;
            if (GRAD) grad[3 * i] = grad[3 * i + 1] = grad[3 * i + 2] = 0.f;
            return;
        }
        const QueryResult q = query_point<ST, GRAD>(m, x, info, qp.strict != 0);
        if (c == 0) {
            sdf[i] = (float)q.sdf;
            valid[i] = q.valid ? 1 : 0;
        }
        if (GRAD && c < 3) grad[3 * i + c] = (float)(c == 0 ? q.grad[0] : c == 1 ? q.grad[1] : q.grad[2]);
    });
}

template <int ST, bool GRAD>
__global__ __launch_bounds__(256) void k_query(const DevMap* __restrict__ pm, QueryParams qp, const float* __restrict__ pts,
                                               int64_t n, float* sdf, uint8_t* valid, float* grad) {
    const DevMap& m = *pm;
    const int c = lane_id() & 3;
    const int64_t stride = (int64_t)gridDim.x * kQueryPoints;
    for (int64_t i = (int64_t)blockIdx.x * kQueryPoints + (threadIdx.x >> 2); i < n; i += stride) {
        double x[3];
        world_point(qp, pts, i, x);
        const QueryResult q = query_point<ST, GRAD>(m, x, home_row(m, x), qp.strict != 0);
        if (c == 0) {
            sdf[i] = (float)q.sdf;
            valid[i] = q.valid ? 1 : 0;
        }
        if (GRAD && c < 3) grad[3 * i + c] = (float)(c == 0 ? q.grad[0] : c == 1 ? q.grad[1] : q.grad[2]);
    }
}

// Backward: per point dL/dx = g_i * d sdf / dx; dL/dp = R^T dL/dx.  Of a point's pose terms lane 0 of the
// group sums dL/dx and lane 1 x cross dL/dx; then per workgroup in a fixed order into FP64 partials.
template <int ST, bool MANY>
__global__ __launch_bounds__(256) void k_query_backward(const DevMap* __restrict__ pm, QueryParams qp, const float* __restrict__ pts,
                                                        int64_t n, const float* __restrict__ gsdf, float* gpts,
                                                        double* partials) {
    const DevMap& m = *pm;
    const int c = lane_id() & 3;
    double acc[3] = {0.0, 0.0, 0.0};
    auto add = [&](int64_t i, const double x[3], uint32_t info) {
        const float gi = gsdf[i];
        const QueryResult q = query_point<ST, true>(m, x, info, qp.strict != 0);
        double g[3] = {0.0, 0.0, 0.0};
        if (q.valid) {
            const double gs = (double)gi;
            for (int k = 0; k < 3; ++k) g[k] = gs * q.grad[k];
        }
        if (c < 3) {
            double v = c == 0 ? g[0] : c == 1 ? g[1] : g[2];
            if (!qp.identity) v = (qp.P.R[0][c] * g[0] + qp.P.R[1][c] * g[1]) + qp.P.R[2][c] * g[2];
            gpts[3 * i + c] = (float)v;
        }
        const double t[3] = {x[1] * g[2] - x[2] * g[1], x[2] * g[0] - x[0] * g[2], x[0] * g[1] - x[1] * g[0]};
        for (int k = 0; k < 3; ++k) acc[k] += c == 0 ? g[k] : t[k];
    };
    if (MANY) {
        uint32_t inf = 0u;  // axes on which a point without a block is not finite: x cross 0 is NaN then
        query_many(m, qp, pts, n, [&](int64_t i, const double x[3], uint32_t info, bool present) {
            if (present) {
                add(i, x, info);
                return;
            }
            gpts[3 * i] = gpts[3 * i + 1] = gpts[3 * i + 2] = 0.f;
            for (int k = 0; k < 3; ++k) inf |= (__builtin_fabs(x[k]) < __builtin_inf() ? 0u : 1u) << k;
        });
        for (int k = 0; k < 3; ++k)
            if (__any((inf & ~(1u << k)) != 0u) && c == 1) acc[k] = __builtin_nan("");
    } else {
        const int64_t stride = (int64_t)gridDim.x * kQueryPoints;
        for (int64_t i = (int64_t)blockIdx.x * kQueryPoints + (threadIdx.x >> 2); i < n; i += stride) {
            double x[3];
            world_point(qp, pts, i, x);
            add(i, x, home_row(m, x));
        }
    }
    __shared__ double red[kQueryPoints][6];
    if (c < 2)
        for (int k = 0; k < 3; ++k) red[threadIdx.x >> 2][3 * c + k] = acc[k];
    __syncthreads();
    if (threadIdx.x < 6) {
        double s = 0.0;
        for (int k = 0; k < kQueryPoints; ++k) s += red[k][threadIdx.x];
        partials[(size_t)blockIdx.x * 6 + threadIdx.x] = s;
    }
}

// Final pose-gradient sum over the workgroup partials, in a fixed order (one workgroup of 256):
// strided per-thread sums, then a tree in LDS.
__global__ __launch_bounds__(256) void k_reduce_partials(const double* __restrict__ partials, int nparts, double* out) {
    __shared__ double red[6][256];
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nparts; b += 256)
        for (int k = 0; k < 6; ++k) s[k] += partials[(size_t)b * 6 + k];
    for (int k = 0; k < 6; ++k) red[k][threadIdx.x] = s[k];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int k = 0; k < 6; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 6) out[threadIdx.x] = red[threadIdx.x][0];
}

static bool make_params(const double* T, int32_t strict, QueryParams& qp) {
    qp.strict = strict;
    if (!T) {
        qp.identity = 1;
        for (int r = 0; r < 3; ++r) {
            for (int c = 0; c < 3; ++c) qp.P.R[r][c] = r == c ? 1.0 : 0.0;
            qp.P.t[r] = 0.0;
        }
        return true;
    }
    qp.identity = 0;
    return pose_from(T, qp.P);
}

}  // namespace mrh

using namespace mrh;

extern "C" mrh_status mrh_query_sdf(mrh_map* map, const float* pts_dev, int64_t n, const double* T_wq, int32_t strict,
                                    float* sdf_dev, uint8_t* valid_dev, float* grad_dev) {
    if (!map || n < 0) return MRH_ERR_INVALID_ARG;
    if (n == 0) return MRH_OK;
    if (!pts_dev || !sdf_dev || !valid_dev) return MRH_ERR_INVALID_ARG;
    QueryParams qp;
    if (!make_params(T_wq, strict, qp)) return set_error(map, MRH_ERR_INVALID_ARG, "non-finite query pose");
    const int64_t per = n >= kQueryMany ? 4 * kQueryWave : kQueryPoints, blocks = (n + per - 1) / per;
    const unsigned grid = (unsigned)(blocks < 65536 ? blocks : 65536);
    launch(map, K_QUERY, [&] {
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, map->stream, map->dmd, qp, pts_dev, n, sdf_dev, valid_dev, grad_dev);
        };
        if (n >= kQueryMany) {
            switch (map->cfg.storage) {
                case MRH_STORE_F16: grad_dev ? go(k_query_many<MRH_STORE_F16, true>) : go(k_query_many<MRH_STORE_F16, false>); break;
                case MRH_STORE_BF16: grad_dev ? go(k_query_many<MRH_STORE_BF16, true>) : go(k_query_many<MRH_STORE_BF16, false>); break;
                default: grad_dev ? go(k_query_many<MRH_STORE_F32, true>) : go(k_query_many<MRH_STORE_F32, false>);
            }
            return;
        }
        switch (map->cfg.storage) {
            case MRH_STORE_F16: grad_dev ? go(k_query<MRH_STORE_F16, true>) : go(k_query<MRH_STORE_F16, false>); break;
            case MRH_STORE_BF16: grad_dev ? go(k_query<MRH_STORE_BF16, true>) : go(k_query<MRH_STORE_BF16, false>); break;
            default: grad_dev ? go(k_query<MRH_STORE_F32, true>) : go(k_query<MRH_STORE_F32, false>);
        }
    });
    return check_hip(map, hipGetLastError(), "query_sdf");
}

extern "C" mrh_status mrh_query_sdf_backward(mrh_map* map, const float* pts_dev, int64_t n, const double* T_wq,
                                             int32_t strict, const float* grad_sdf_dev, float* grad_pts_dev,
                                             double grad_pose_host[6]) {
    if (!map || n < 0 || !grad_pose_host) return MRH_ERR_INVALID_ARG;
    if (n > 0 && (!pts_dev || !grad_sdf_dev || !grad_pts_dev)) return MRH_ERR_INVALID_ARG;
    QueryParams qp;
    if (!make_params(T_wq, strict, qp)) return set_error(map, MRH_ERR_INVALID_ARG, "non-finite query pose");
    for (int k = 0; k < 6; ++k) grad_pose_host[k] = 0.0;
    if (n == 0) return MRH_OK;
    const bool many = n >= kAdjointMany;
    const int64_t per = many ? 4 * kQueryWave : kQueryPoints, blocks = (n + per - 1) / per;
    const int grid = (int)(blocks < map->partials_cap ? blocks : map->partials_cap);
    launch(map, K_QUERY_BACKWARD, [&] {
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, map->stream, map->dmd, qp, pts_dev, n, grad_sdf_dev, grad_pts_dev, map->partials);
        };
        switch (map->cfg.storage) {
            case MRH_STORE_F16: many ? go(k_query_backward<MRH_STORE_F16, true>) : go(k_query_backward<MRH_STORE_F16, false>); break;
            case MRH_STORE_BF16: many ? go(k_query_backward<MRH_STORE_BF16, true>) : go(k_query_backward<MRH_STORE_BF16, false>); break;
            default: many ? go(k_query_backward<MRH_STORE_F32, true>) : go(k_query_backward<MRH_STORE_F32, false>);
        }
    });
    launch(map, K_REDUCE, [&] {
        hipLaunchKernelGGL(k_reduce_partials, dim3(1), dim3(256), 0, map->stream, map->partials, grid, map->pose_out);
    });
    mrh_status st = check_hip(map, hipGetLastError(), "query_sdf_backward");
    if (st != MRH_OK) return st;
    st = check_hip(map, hipMemcpyAsync(grad_pose_host, map->pose_out, 48, hipMemcpyDeviceToHost, map->stream),
                   "query_sdf_backward");
    if (st != MRH_OK) return st;
    return check_hip(map, hipStreamSynchronize(map->stream), "query_sdf_backward");
}
