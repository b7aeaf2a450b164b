// LiDAR fusion of one map (Sec. 3.1 "3D Point Cloud", Eq. 1; Eq. 3, Eq. 5; Sec. 3.2.1).
//
// One scan is four launches on the map's stream: k_alloc_points (its last workgroups also run the
// allocation-side frame hand-off), k_rays, k_touch_queue (the touched blocks onto the per-level
// update queues) and k_apply_points (update tasks over those queues; the first workgroups also run
// the update-side hand-off).
#include <cmath>
#include <type_traits>

#include "mrh_points.h"

namespace mrh {

__global__ __launch_bounds__(256) void k_alloc_points(const DevMap* __restrict__ pm, ScanParams sp) {
    const uint32_t parts = duty_parts(gridDim.x), part = gridDim.x - 1u - blockIdx.x;
    if (part < parts) alloc_duties(*pm, sp.parity, part, parts);
    points_alloc_chunk(*pm, sp, blockIdx.x);
}

template <bool WIDE>
__global__ __launch_bounds__(256) void k_rays(const DevMap* __restrict__ pm, ScanParams sp) {
    __shared__ RayLds lds;
    points_ray_chunk<WIDE>(*pm, sp, blockIdx.x, lds);
}

// After the ray launch: the touched blocks onto the update queues (workgroup w takes block ids
// w * 256 * kTouchPerThread onwards).
__global__ __launch_bounds__(256) void k_touch_queue(const DevMap* __restrict__ pm, int par) {
    const DevMap& m = *pm;
    const uint32_t nb = min(m.ctr->n_blocks, m.max_blocks);
    const uint32_t per = blockDim.x * (uint32_t)kTouchPerThread;
    for (uint32_t first = blockIdx.x * per; first < nb; first += gridDim.x * per)
        queue_touched(m, first, min(per, nb - first), par);
}

template <int ST, bool WIDE>
__global__ __launch_bounds__(256) void k_apply_points(const DevMap* __restrict__ pm, int par) {
    const DevMap& m = *pm;
    if (blockIdx.x < duty_parts(gridDim.x)) update_duties(m, par, blockIdx.x, duty_parts(gridDim.x));
    const uint32_t wave = uniform((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const uint32_t nwaves = (gridDim.x * blockDim.x) >> 6;
    const TaskCounts n = frame_task_counts(m, false, par);
    const uint32_t ntask = points_task_count(n);
    // merges of level-0 / level-1 blocks are recorded and done in batches (see run_deferred)
    __shared__ uint32_t dbuf[4][4 * kDefer];
    __shared__ ApplyLds lds[4];
    const uint32_t wv = uniform(threadIdx.x >> 6);
    DeferList dl{dbuf[wv], 0u};
    unsigned long long m0 = 0, m1 = 0;
    TaskStats as;
    for (uint32_t t = wave; t < ntask; t += nwaves) {
        as.add(points_update_task<ST, WIDE>(m, t, n, par, &dl, lds[wv]));
        if (!dl.ready(kApplyBlocks)) run_deferred<ST>(m, dl, par, m0, m1);
    }
    run_deferred<ST>(m, dl, par, m0, m1);
    as.merge0 += m0;
    as.merge1 += m1;
    flush_task_stats(m, as, false);
}

// Rays per workgroup of a scan's allocation and ray launches.  The ray launch's LDS tables gain from many rays,
// but below some eight workgroups per CU a launch lasts as long as one of them.  Ray launch: 8000 rays 190 us by
// 16, 146 by 4, 162 by 2; 31713 rays 366 by 16, 324 by 8, 349 by 4; 131072 rays 508 by 16, 522 by 8.
// Allocation, mean of three scans: 8000 rays 63 us by 16, 49 by 4; 31713 rays 93 by 16, 85 by 8.  Without carving a
// ray has a few blocks only, of which 16 rays just fill a wave: 8000 rays on a street 24 + 27 us (allocation
// and rays of the first scan) by 4, 14 + 17 by 16; 31713 rays 33 + 50 by 8, 26 + 39 by 16.  (A batch's scans
// share the chip: always kRaysPerGroup.)
static int32_t rays_per_group(const mrh_map* map, int64_t n) {
    if (!map->cfg.carve) return kRaysPerGroup;
    return n < (1 << 14) ? 4 : (n < (1 << 16) ? 8 : kRaysPerGroup);
}

// Blocks a ray's walk can visit: the guard of the block walk bounds it by 4 + the sum over the
// axes of the cells the segment spans (carving: up to max_range + tau long; otherwise 2 tau).
static int32_t ray_block_cap(const mrh_config& c) {
    const double len = c.carve ? c.max_range + c.tau : 2.0 * c.tau;
    const double cells = 1.7320508075688772 * len / (8.0 * c.voxel) + 8.0;
    return cells < 1024.0 ? (int32_t)cells : 1024;
}

// LiDAR state of a map: accumulators (first scan) and per-ray block-key buffers for n rays.
mrh_status ensure_lidar(mrh_map* map, int64_t n) {
    DevMap& d = map->dm;
    mrh_status st = MRH_OK;
    bool changed = false;
    auto alloc = [&](void* at, size_t bytes, const char* what) {  // at: the address of a pointer
        void** p = (void**)at;
        changed = true;
        if (st != MRH_OK || *p) return;  // (there since a call that ran out of memory further on)
        st = check_hip(map, hipMalloc(p, bytes), what);
        if (st != MRH_OK) *p = nullptr;
        else if ((st = check_hip(map, hipMemsetAsync(*p, 0, bytes, map->stream), what)) != MRH_OK) {
            (void)hipFree(*p);
            *p = nullptr;
        }
    };
    if (!map->lidar_ready) {
        alloc(&d.btouch, (size_t)d.max_blocks * 8, "touch masks");
        for (int l = 0; l < map->cfg.levels; ++l) {
            const size_t nv = (size_t)d.heap_cap[l] * (size_t)(side_of(l) * side_of(l) * side_of(l));
            alloc(&d.acc_sat[l], nv * 4, "scan accumulators");
            alloc(&d.acc_s1[l], nv * 8, "scan accumulators");
            alloc(&d.acc_s2[l], nv * 8, "scan accumulators");
        }
        d.band_bias = (long long)std::ceil(map->cfg.tau * kS1Scale) + 1;
        d.rcap_k = ray_block_cap(map->cfg);
        if (st == MRH_OK) map->lidar_ready = true;
    }
    // A ray's walk enters each cell of its lattice once, so a voxel takes at most n observations, each of up to
    // 2 bias in the shared word and bias^2 in the squares: with fewer than 2^20 of them, and their sums below
    // 2^44 and 2^64 (n tau < 2^19 m, n tau^2 < 2^16 m^2), every voxel's words hold.  Larger scans and
    // truncations keep their counts, or the squares' halves, apart.
    auto words = [&](auto planes, size_t size) {
        for (int l = 0; l < map->cfg.levels; ++l)
            alloc(&planes[l], (size_t)d.heap_cap[l] * (size_t)(side_of(l) * side_of(l) * side_of(l)) * size, "scan accumulators");
        return st == MRH_OK ? 1 : 0;
    };
    const double bias = (double)d.band_bias;
    if (st == MRH_OK && !d.band_wide && ((double)n >= 0x1p20 || (double)n * 2.0 * bias >= 0x1p44)) d.band_wide = words(d.acc_band, 4);
    if (st == MRH_OK && !d.square_wide && (double)n * bias * bias >= 0x1p64) d.square_wide = words(d.acc_s2h, 8);
    if (st == MRH_OK && n > map->rcap_n) {
        st = check_hip(map, hipStreamSynchronize(map->stream), "ray buffers");
        if (d.rslots) (void)hipFree(plain(d.rslots));
        if (d.rcount) (void)hipFree(plain(d.rcount));
        d.rslots = nullptr;
        d.rcount = nullptr;
        map->rcap_n = 0;
        alloc(&d.rslots, (size_t)n * (size_t)d.rcap_k * 4, "ray block slots");
        alloc(&d.rcount, (size_t)n * 4, "ray block counts");
        if (st == MRH_OK) map->rcap_n = n;
    }
    if (st == MRH_OK && changed) st = upload_descriptor(map);
    return st;
}

}  // namespace mrh

using namespace mrh;

extern "C" mrh_status mrh_integrate_points(mrh_map* map, const float* xyz_dev, int64_t n, const double T_ws[16]) {
    if (!map || !T_ws || n < 0 || (n > 0 && !xyz_dev)) return MRH_ERR_INVALID_ARG;
    if (map->cfg.color) return set_error(map, MRH_ERR_INVALID_ARG, "a map with colour fuses RGB-D frames only");
    ScanParams sp;
    if (!pose_from(T_ws, sp.P)) return set_error(map, MRH_ERR_INVALID_ARG, "non-finite pose");
    sp.xyz = global(xyz_dev);
    sp.n = n;
    sp.rays = rays_per_group(map, n);
    mrh_status st = ensure_lidar(map, n);
    if (st != MRH_OK) return st;
    sp.parity = (int32_t)(map->frames & 1u);
    map->frames += 1;
    const int par = sp.parity;
    // the allocation and update launches always run (they carry the frame hand-off); the ray launch has the
    // allocation's workgroups
    const unsigned agrid = n > 0 ? (unsigned)((n + sp.rays - 1) / sp.rays) : 1u;
    launch(map, K_ALLOC_POINTS,
           [&] { hipLaunchKernelGGL(k_alloc_points, dim3(agrid), dim3(256), 0, map->stream, map->dmd, sp); });
    auto rest = [&](auto w) {
        constexpr bool WIDE = decltype(w)::value;
        if (n > 0) {
            launch(map, K_RAYS, [&] {
                hipLaunchKernelGGL(k_rays<WIDE>, dim3(agrid), dim3(256), 0, map->stream, map->dmd, sp);
                hipLaunchKernelGGL(k_touch_queue, dim3(1024), dim3(256), 0, map->stream, map->dmd, par);
            });
        }
        launch(map, K_APPLY_POINTS, [&] {
            const dim3 g(1024), b(256);
            switch (map->cfg.storage) {
                case MRH_STORE_F16: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_apply_points<MRH_STORE_F16, WIDE>), g, b, 0, map->stream, map->dmd, par); break;
                case MRH_STORE_BF16: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_apply_points<MRH_STORE_BF16, WIDE>), g, b, 0, map->stream, map->dmd, par); break;
                default: hipLaunchKernelGGL(HIP_KERNEL_NAME(k_apply_points<MRH_STORE_F32, WIDE>), g, b, 0, map->stream, map->dmd, par);
            }
        });
    };
    if (map->dm.square_wide) rest(std::true_type());
    else rest(std::false_type());
    return check_hip(map, hipGetLastError(), "integrate_points");
}

extern "C" mrh_status mrh_integrate_points_sequence(mrh_map* map, const float* xyz_dev, int32_t n_frames, int64_t n,
                                                    const double* T_ws) {
    if (!map || !T_ws || n_frames < 0 || n < 0 || (n > 0 && !xyz_dev)) return MRH_ERR_INVALID_ARG;
    Pose P;
    for (int32_t k = 0; k < n_frames; ++k)
        if (!pose_from(T_ws + 16 * k, P)) return set_error(map, MRH_ERR_INVALID_ARG, "scan %d: non-finite pose", k);
    for (int32_t k = 0; k < n_frames; ++k) {
        const mrh_status st = mrh_integrate_points(map, xyz_dev + (size_t)3 * (size_t)n * (size_t)k, n, T_ws + 16 * k);
        if (st != MRH_OK) return st;
    }
    return MRH_OK;
}
