// Colours of RGB-D frames (Sec. 3: a voxel stores a colour): entry point and extraction.
//
// A voxel that a frame updates averages the RGB value of its pixel into its colour,
// C <- C + (c - C) / W with the weight W after the update (Eq. 3 with w = 1).  The update launch does so
// with the state (integrate_fine_block and its siblings): it has the voxel's pixel, decision and weight
// at hand, which a launch of its own took again at the price of the update (640 x 480 room frames:
// update and colour launches 27.2 + 28.6 us, together 30.8).  A block that merges one level coarser pools
// its colours as the weighted mean of the observed children, as the TSDF is; new blocks cannot merge in
// their first frame (no voxel reaches min_obs >= 2 observations).

#include "mrh_depth.h"

namespace mrh {

// Colours out, in the voxel order of mrh_extract_blocks (x fastest per block) and its manner: lanes
// follow the output's floats, so that the stores fill whole lines (room map at 1 cm: 75 -> 38 us).
__global__ __launch_bounds__(256) void k_extract_color(const DevMap* __restrict__ pm, const ExtractRow* __restrict__ rows,
                                                       uint32_t nrows, float* __restrict__ out) {
    const DevMap& m = *pm;
    const int lane = threadIdx.x & 63, v = lane & 7, wave = (int)uniform(threadIdx.x >> 6);
    for (uint32_t first = blockIdx.x * kExtractRows; first < nrows; first += gridDim.x * kExtractRows) {
        const uint32_t row = first + (lane >> 3);
        ExtractRow e{0, 0u, kNoBlockBit};
        if (row < nrows) e = rows[row];
        const bool block = !(e.info & kNoBlockBit);
        const int lvl = (int)((e.info >> kLevelShift) & 3u);
        // (the order of the eight voxels of a level-2 block is the same in both)
        if (wave == 0 && block && (lvl == 2 || (lvl == 3 && v == 0))) {
            const float MRH_GLOBAL* c = lvl == 2 ? m.C[2] + 24 * (size_t)(e.info & kSlotMask) : m.C[3] + 3 * (size_t)(e.info & kSlotMask);
            for (int ch = 0; ch < 3; ++ch) out[3 * (e.off + v) + ch] = c[3 * v + ch];
        }
        unsigned long long large = __ballot(block && lvl < 2 && v == 0);
        for (int turn = 0; large; ++turn) {
            const int src = __ffsll((long long)large) - 1;
            large &= large - 1;
            if ((turn & 3) != wave) continue;
            const uint32_t info = (uint32_t)uniform(__shfl((int)e.info, src));
            const int64_t off = (int64_t)((unsigned long long)(uint32_t)uniform(__shfl((int)(uint32_t)((unsigned long long)e.off >> 32), src)) << 32 |
                                          (uint32_t)uniform(__shfl((int)(uint32_t)(unsigned long long)e.off, src)));
            float* o = out + 3 * off + lane;
            if (((info >> kLevelShift) & 3u) == 1u) {
                const float MRH_GLOBAL* c = m.C[1] + 192 * (size_t)(info & kSlotMask);
                for (int k = 0; k < 3; ++k) {
                    const int q = lane + 64 * k, x = q / 3;
                    const uint32_t p = spread3(x & 3) | spread3((x >> 2) & 3) << 1 | spread3(x >> 4) << 2;
                    o[64 * k] = c[3 * p + (uint32_t)(q - 3 * x)];
                }
            } else {
                const float MRH_GLOBAL* c = m.C[0] + 1536 * (size_t)(info & kSlotMask);
                float f[24];
#pragma unroll
                for (int k = 0; k < 24; ++k) {
                    const int q = lane + 64 * k, x = q / 3;
                    const uint32_t p = spread3(x & 7) | spread3((x >> 3) & 7) << 1 | spread3(x >> 6) << 2;
                    f[k] = c[3 * p + (uint32_t)(q - 3 * x)];
                }
#pragma unroll
                for (int k = 0; k < 24; ++k) o[64 * k] = f[k];
            }
        }
    }
}

}  // namespace mrh

using namespace mrh;

extern "C" mrh_status mrh_integrate_rgbd(mrh_map* map, const float* depth_dev, const uint8_t* rgb_dev, int32_t width,
                                         int32_t height, const double K[4], const double T_ws[16]) {
    if (!map || !rgb_dev) return MRH_ERR_INVALID_ARG;
    if (!map->cfg.color) return set_error(map, MRH_ERR_INVALID_ARG, "the map was created without colour");
    return integrate_depth_frame(map, depth_dev, rgb_dev, width, height, K, T_ws);
}

extern "C" mrh_status mrh_extract_color(mrh_map* map, float* rgb_dev, int64_t voxel_cap, int64_t* n_voxels) {
    if (!map || !n_voxels) return MRH_ERR_INVALID_ARG;
    if (!map->cfg.color) return set_error(map, MRH_ERR_INVALID_ARG, "the map was created without colour");
    uint32_t nout = 0;
    int64_t nvox = 0;
    mrh_status st = scan_rows(map, "extract colour", nout, nvox);
    if (st != MRH_OK) return st;
    *n_voxels = nvox;
    if (!rgb_dev) return MRH_OK;
    if (voxel_cap < nvox) return set_error(map, MRH_ERR_BUFFER_TOO_SMALL, "colour needs %lld voxels", (long long)nvox);
    if (nout == 0) return MRH_OK;
    hipLaunchKernelGGL(k_extract_color, dim3(extract_grid(nout)), dim3(256), 0, map->stream,
                       map->dmd, map->extract_rows, nout, rgb_dev);
    st = check_hip(map, hipGetLastError(), "extract colour");
    if (st == MRH_OK) st = check_hip(map, hipStreamSynchronize(map->stream), "extract colour");
    return st;
}
