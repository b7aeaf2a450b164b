// Map lifetime, reset, statistics, extraction and error reporting.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include "mrh_update.h"

namespace mrh {

mrh_status set_error(mrh_map* m, mrh_status code, const char* fmt, ...) {
    if (m) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(m->err, sizeof(m->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

mrh_status check_hip(mrh_map* m, hipError_t e, const char* what) {
    if (e == hipSuccess) return MRH_OK;
    (void)hipGetLastError();  // reported here: the next launch's check would find it again
    return set_error(m, e == hipErrorOutOfMemory ? MRH_ERR_OOM : MRH_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// Kernels read the map descriptor through a pointer: a ~900-byte by-value argument would not fit
// the scalar register file and would be spilled into vector lanes on every launch.
mrh_status upload_descriptor(mrh_map* m) {
    ++m->dm_version;
    mrh_status st = check_hip(m, hipMemcpyAsync(m->dmd, &m->dm, sizeof(DevMap), hipMemcpyHostToDevice, m->stream),
                              "descriptor upload");
    if (st == MRH_OK) st = check_hip(m, hipStreamSynchronize(m->stream), "descriptor upload");
    return st;
}

bool pose_from(const double* T, Pose& P) {
    if (!T) return false;
    for (int i = 0; i < 16; ++i)
        if (!std::isfinite(T[i])) return false;
    for (int r = 0; r < 3; ++r) {
        for (int c = 0; c < 3; ++c) P.R[r][c] = T[4 * r + c];
        P.t[r] = T[4 * r + 3];
    }
    return true;
}

// Empty table, full free stacks, zero counters.
__global__ void k_reset(const DevMap* __restrict__ pm, uint32_t n_hash) {
    const DevMap& m = *pm;
    const uint32_t tid = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    for (uint32_t i = tid; i < n_hash; i += stride) store_as(m.table + i, u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, kInvalidId, kNoBlockBit});  // kEmptyKey
    for (int n = 0; n < m.levels; ++n) {
        const uint32_t cap = (uint32_t)m.heap_cap[n];
        for (uint32_t i = tid; i < cap; i += stride) m.stack[n][i] = cap - 1 - i;  // pops give 0, 1, 2, ...
    }
    if (tid == 0) {
        DevCounters MRH_GLOBAL* c = m.ctr;
        c->n_blocks = 0;
        c->pops0 = 0;
        c->error_flags.v = 0;
        for (int p = 0; p < 2; ++p) {
            c->n_prev[p] = 0;
            c->pending0[p].v = 0;
            for (int n = 0; n < 4; ++n) c->vis_n[p][n].v = 0;
            c->duty[p].v = 0;
        }
        for (int n = 0; n < 4; ++n) {
            c->top[n].v = n < m.levels ? m.heap_cap[n] : 0;
            c->pending[n].v = 0;
        }
    }
    if (tid < 16 * kStripes) m.ctr->frame[tid >> 4][tid & 15] = 0;
}

// Rows of an extraction: the blocks in table order without those streamed out to the host store, and
// the sum of the voxels before each.  Two launches over chunks of kExtractChunk ids, as far as blocks have been
// handed out: sums, then rows (for each chunk the sums before it are added up).  Against a copy of every descriptor to the host, a
// loop over them there and two uploads into new allocations.
__device__ inline unsigned long long row_weight(uint32_t info) {  // rows << 40 | voxels
    if (info & kGoneBit) return 0ull;
    const int b = 3 * (3 - (int)((info >> kLevelShift) & 3u));
    return 1ull << 40 | ((info & kNoBlockBit) ? 0ull : 1ull << b);
}

__host__ __device__ inline uint32_t extract_chunks(uint32_t blocks) { return (blocks + kExtractChunk - 1) / kExtractChunk; }

__device__ inline uint32_t block_count(const DevMap& m) {
    const uint32_t n = m.ctr->n_blocks;
    return n < m.max_blocks ? n : m.max_blocks;
}

__global__ __launch_bounds__(256) void k_extract_sums(const DevMap* __restrict__ pm, ExtractRow* __restrict__ rows) {
    const DevMap& m = *pm;
    const uint32_t nb = block_count(m);
    __shared__ uint32_t part[4][2];
    for (uint32_t chunk = blockIdx.x; chunk < extract_chunks(nb); chunk += gridDim.x) {
        unsigned long long n = 0;
#pragma unroll
        for (uint32_t k = 0; k < kExtractChunk / 256; ++k) {
            const uint32_t id = chunk * kExtractChunk + k * 256 + threadIdx.x;
            n += id < nb ? row_weight(m.binfo[id]) : 0ull;
        }
        uint32_t r = (uint32_t)(n >> 40), v = (uint32_t)n;  // (a chunk has at most 2^20 voxels)
        static_assert(kExtractChunk * 512ull < (1ull << 32), "chunk sums in 32 bits");
        for (int o = 1; o < 64; o <<= 1) r += (uint32_t)__shfl_xor((int)r, o), v += (uint32_t)__shfl_xor((int)v, o);
        if ((threadIdx.x & 63u) == 0) part[threadIdx.x >> 6][0] = r, part[threadIdx.x >> 6][1] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < 4; ++w) r += part[w][0], v += part[w][1];
            rows[m.max_blocks + chunk] = ExtractRow{(int64_t)v, r, 0u};
        }
        __syncthreads();
    }
}

// total: where the number of rows and of voxels goes.
__global__ __launch_bounds__(256) void k_extract_rows(const DevMap* __restrict__ pm, ExtractRow* __restrict__ rows,
                                                      ExtractRow* __restrict__ total) {
    const DevMap& m = *pm;
    const uint32_t nb = block_count(m), t = threadIdx.x, chunks = extract_chunks(nb);
    const ExtractRow* const sums = rows + m.max_blocks;
    __shared__ unsigned long long vbase[256];
    __shared__ uint32_t rbase[256];
    if (nb == 0 && blockIdx.x == 0 && t == 0) *total = ExtractRow{0, 0u, 0u};
    for (uint32_t chunk = blockIdx.x; chunk < chunks; chunk += gridDim.x) {
        const uint32_t id0 = chunk * kExtractChunk + t * (kExtractChunk / 256);
        // the chunks before this one, with this one's threads on top
        unsigned long long v = 0;
        uint32_t r = 0;
        for (uint32_t i = t; i < chunk; i += 256) v += (unsigned long long)sums[i].off, r += sums[i].id;
        vbase[t] = v;
        rbase[t] = r;
        __syncthreads();
        for (uint32_t o = 128; o; o >>= 1) {
            if (t < o) vbase[t] += vbase[t + o], rbase[t] += rbase[t + o];
            __syncthreads();
        }
        const unsigned long long v0 = vbase[0];
        const uint32_t r0 = rbase[0];
        uint32_t info[kExtractChunk / 256];
        unsigned long long own = 0;
#pragma unroll
        for (uint32_t k = 0; k < kExtractChunk / 256; ++k) {
            info[k] = id0 + k < nb ? m.binfo[id0 + k] : kGoneBit;
            own += row_weight(info[k]);
        }
        __syncthreads();
        vbase[t] = own & ((1ull << 40) - 1ull);
        rbase[t] = (uint32_t)(own >> 40);
        __syncthreads();
        for (uint32_t o = 1; o < 256; o <<= 1) {
            const unsigned long long a = t >= o ? vbase[t - o] : 0ull;
            const uint32_t b = t >= o ? rbase[t - o] : 0u;
            __syncthreads();
            vbase[t] += a;
            rbase[t] += b;
            __syncthreads();
        }
        v = v0 + (t ? vbase[t - 1] : 0ull);
        r = r0 + (t ? rbase[t - 1] : 0u);
#pragma unroll
        for (uint32_t k = 0; k < kExtractChunk / 256; ++k) {
            const unsigned long long w = row_weight(info[k]);
            if (w) rows[r] = ExtractRow{(int64_t)v, id0 + k, info[k]};
            r += (uint32_t)(w >> 40);
            v += w & ((1ull << 40) - 1ull);
        }
        if (chunk == chunks - 1 && t == 255) *total = ExtractRow{(int64_t)v, r, 0u};
        __syncthreads();
    }
}

// Copy blocks out: keys, levels and (optionally) voxels from Morton to x-fastest order.  A workgroup takes
// kExtractRows rows and reads their entries together; its first wave copies all voxels of those of levels
// 2 and 3 at once, and the waves share the larger blocks.  Lanes follow the output, whose rows the stores then fill whole; the
// Morton-ordered reads stay within the block's 4 KB.  Lanes in Morton order wrote 16-byte pieces: bf16 street map
// of 31 x 1023 rays 900 -> 345 us, room map at 1 cm 58 -> 28 us, f16 room at 2 cm 16.6 -> 10 us.
template <int ST>
__global__ __launch_bounds__(256) void k_extract(const DevMap* __restrict__ pm, const ExtractRow* __restrict__ rows, uint32_t nrows,
                                                 int32_t* __restrict__ keys, uint8_t* __restrict__ levels,
                                                 int64_t* __restrict__ offsets, float* __restrict__ D,
                                                 uint32_t* __restrict__ W, float* __restrict__ S2) {
    const DevMap& m = *pm;
    const int lane = threadIdx.x & 63, v = lane & 7, wave = (int)uniform(threadIdx.x >> 6);
    static_assert(kExtractRows * 8 == 64, "eight lanes per row");
    for (uint32_t first = blockIdx.x * kExtractRows; first < nrows; first += gridDim.x * kExtractRows) {
        const uint32_t row = first + (lane >> 3);
        ExtractRow e{0, 0u, kNoBlockBit};
        if (row < nrows) e = rows[row];
        if (wave == 0 && row < nrows) {
            const int lvl = (int)((e.info >> kLevelShift) & 3u);
            if (v == 0) {
                if (keys) {
                    int32_t x, y, z;
                    unpack_key(m.bkey[e.id], x, y, z);
                    keys[3 * (size_t)row] = x;
                    keys[3 * (size_t)row + 1] = y;
                    keys[3 * (size_t)row + 2] = z;
                }
                if (levels) levels[row] = (e.info & kNoBlockBit) ? 0xFF : (uint8_t)lvl;
                if (offsets) offsets[row] = e.off;
            }
            if (v == 1 && offsets && row == nrows - 1)
                offsets[nrows] = e.off + (int64_t)(row_weight(e.info) & ((1ull << 40) - 1ull));
        }
        if (!(D || W || S2)) continue;
        const bool block = !(e.info & kNoBlockBit);
        const int lvl = (int)((e.info >> kLevelShift) & 3u);
        auto out = [&](int64_t o, float d, uint32_t w, float s2) {
            if (D) D[o] = d;
            if (W) W[o] = w;
            if (S2) S2[o] = s2;
        };
        // (the order of the eight voxels of a level-2 block is the same in both)
        float d, s2;
        uint32_t w;
        if (wave == 0 && block && lvl == 2) {
            Store<ST>::get(m, 2, (size_t)(e.info & kSlotMask) * 8 + v, d, w, s2);
            out(e.off + v, d, w, s2);
        } else if (wave == 0 && block && lvl == 3 && v == 0) {
            Store<ST>::get(m, 3, (size_t)(e.info & kSlotMask), d, w, s2);
            out(e.off, d, w, s2);
        }
        unsigned long long large = __ballot(block && lvl < 2 && v == 0);
        for (int turn = 0; large; ++turn) {
            const int src = __ffsll((long long)large) - 1;
            large &= large - 1;
            if ((turn & 3) != wave) continue;
            const uint32_t info = (uint32_t)uniform(__shfl((int)e.info, src));
            const int64_t off = (int64_t)((unsigned long long)(uint32_t)uniform(__shfl((int)(uint32_t)((unsigned long long)e.off >> 32), src)) << 32 |
                                          (uint32_t)uniform(__shfl((int)(uint32_t)(unsigned long long)e.off, src)));
            if (((info >> kLevelShift) & 3u) == 1u) {
                const uint32_t p = spread3(lane & 3) | spread3((lane >> 2) & 3) << 1 | spread3(lane >> 4) << 2;
                Store<ST>::get(m, 1, (size_t)(info & kSlotMask) * 64 + p, d, w, s2);
                out(off + lane, d, w, s2);
            } else {
                const uint32_t p = spread3(lane & 7) | spread3(lane >> 3) << 1;
                const size_t base = (size_t)(info & kSlotMask) * 512 + p;
                float dd[8], ss[8];
                uint32_t ww[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) Store<ST>::get(m, 0, base + (spread3(k) << 2), dd[k], ww[k], ss[k]);
#pragma unroll
                for (int k = 0; k < 8; ++k) out(off + lane + 64 * k, dd[k], ww[k], ss[k]);
            }
        }
    }
}

mrh_status scan_rows(mrh_map* m, const char* what, uint32_t& rows, int64_t& voxels) {
    const uint32_t chunks = extract_chunks(m->dm.max_blocks), grid = chunks < kExtractGrid ? chunks : kExtractGrid;
    mrh_status st = MRH_OK;
    if (!m->extract_rows)
        st = check_hip(m, hipMalloc((void**)&m->extract_rows, ((size_t)m->dm.max_blocks + chunks + 1) * sizeof(ExtractRow)), what);
    if (st != MRH_OK) return st;
    ExtractRow* const end = m->extract_rows + m->dm.max_blocks + chunks;
    hipLaunchKernelGGL(k_extract_sums, dim3(grid), dim3(256), 0, m->stream, m->dmd, m->extract_rows);
    hipLaunchKernelGGL(k_extract_rows, dim3(grid), dim3(256), 0, m->stream, m->dmd, m->extract_rows, end);
    st = check_hip(m, hipGetLastError(), what);
    ExtractRow total{};
    if (st == MRH_OK)
        st = check_hip(m, hipMemcpyAsync(&total, end, sizeof(total), hipMemcpyDeviceToHost, m->stream), what);
    if (st == MRH_OK) st = check_hip(m, hipStreamSynchronize(m->stream), what);
    rows = total.id;
    voxels = total.off;
    return st;
}

}  // namespace mrh

using namespace mrh;

extern "C" {

int32_t mrh_abi_version(void) { return MRH_ABI_VERSION; }

uint32_t mrh_block_hash(int32_t x, int32_t y, int32_t z, uint64_t n_hash) {
    if (n_hash == 0) return 0;
    return (uint32_t)((uint64_t)spatial_hash(x, y, z) % n_hash);
}

const char* mrh_last_error(const mrh_map* map) { return map ? map->err : "null map"; }

static void free_all(mrh_map* m) {
    stream_free(m);
    DevMap& d = m->dm;
    void* ptrs[] = {plain(d.table), plain(d.bslot), plain(d.bkey), plain(d.binfo), plain(d.bvsum), plain(d.bvcnt), m->ctr, m->partials, m->pose_out, m->dmd,
                    m->count_dev, m->mesh_order, m->extract_rows};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    if (d.btouch) (void)hipFree(plain(d.btouch));
    for (int p = 0; p < 2; ++p)
        if (d.pend0[p]) (void)hipFree(plain(d.pend0[p]));
    if (d.rslots) (void)hipFree(plain(d.rslots));
    if (d.rcount) (void)hipFree(plain(d.rcount));
    if (m->tile_max) (void)hipFree(m->tile_max);
    for (int n = 0; n < 4; ++n)
        if (d.vis[n]) (void)hipFree(plain(d.vis[n]));
    for (int n = 0; n < 2; ++n)
        if (d.vrect[n]) (void)hipFree(plain(d.vrect[n]));
    for (int n = 0; n < 4; ++n) {
        void* lp[] = {plain(d.stack[n]), plain(d.pend[n]), plain(d.DW[n]), plain(d.S2[n]), plain(d.C[n]), plain(d.acc_sat[n]), plain(d.acc_band[n]), plain(d.acc_s1[n]), plain(d.acc_s2[n]), plain(d.acc_s2h[n])};
        for (void* p : lp)
            if (p) (void)hipFree(p);
    }
}

mrh_status mrh_map_create(const mrh_config* cfg, void* stream, mrh_map** out) {
    if (!cfg || !out) return MRH_ERR_INVALID_ARG;
    *out = nullptr;
    const mrh_config& c = *cfg;
    const bool pow2 = c.hash_slots > 0 && (c.hash_slots & (c.hash_slots - 1)) == 0;
    if (!(c.voxel > 0.0) || !std::isfinite(c.voxel) || c.levels < 1 || c.levels > 4 || !(c.tau > 0.0) ||
        c.min_obs < 1 || !pow2 || c.max_blocks < 1 || c.hash_slots < 2 * c.max_blocks ||
        c.hash_slots > (int64_t(1) << 31) || c.max_blocks > (int64_t(1) << 30) || !(c.var_thr >= 0.0) ||
        c.storage < MRH_STORE_F32 || c.storage > MRH_STORE_BF16 || c.form < 0 || c.form > 1 || c.color < 0 ||
        c.color > 1 || (c.color && c.min_obs < 2))
        return MRH_ERR_INVALID_ARG;
    for (int n = 0; n < 4; ++n)
        if (c.heap_blocks[n] < 0 || c.heap_blocks[n] > (int64_t)kSlotMask + 1) return MRH_ERR_INVALID_ARG;

    mrh_map* m = new mrh_map();
    m->cfg = c;
    m->stream = (hipStream_t)stream;
    if (hipGetDevice(&m->device) != hipSuccess) {
        delete m;
        return MRH_ERR_HIP;
    }
    DevMap& d = m->dm;
    d.hmask = (uint32_t)(c.hash_slots - 1);
    d.max_probe = c.max_probe > 0 ? c.max_probe : 4096;
    d.max_blocks = (uint32_t)c.max_blocks;
    d.levels = c.levels;
    d.B = 8.0 * c.voxel;
    d.invB = 1.0 / d.B;
    for (int n = 0; n < 4; ++n) {
        d.nu[n] = c.voxel * (double)(1 << n);
        d.inv_nu[n] = 1.0 / d.nu[n];
    }
    d.tau = c.tau;
    d.tau_f = (float)c.tau;
    d.inv_tau_f = (float)(1.0 / c.tau);
    d.tau2_f = (float)(c.tau * c.tau);
    {
        float mf = (float)c.max_depth;
        if ((double)mf > c.max_depth) mf = std::nextafter(mf, -INFINITY);
        if (std::isnan(c.max_depth)) mf = -1.f;  // no depth is <= a maximum that is not a number
        d.max_depth_f = mf;
    }
    d.var_thr = c.var_thr;
    d.max_depth = c.max_depth;
    d.r2lo = c.min_range * c.min_range;
    d.r2hi = c.max_range * c.max_range;
    d.min_obs = c.min_obs;
    d.form = c.form;
    d.carve = c.carve;
    d.storage = c.storage;

    mrh_status st = MRH_OK;
    auto alloc = [&](void* p, size_t bytes, const char* what) {  // p: the address of a pointer
        if (st != MRH_OK) return;
        st = check_hip(m, hipMalloc((void**)p, bytes ? bytes : 16), what);
    };
    const size_t nh = (size_t)c.hash_slots, nb = (size_t)c.max_blocks;
    alloc(&d.table, nh * sizeof(HashSlot), "hash table");
    alloc(&d.bslot, nb * 4, "block hash slots");
    alloc(&d.bkey, nb * 8, "block keys");
    alloc(&d.binfo, nb * 4, "block info");
    alloc(&d.bvsum, nb * 8, "block variance sums");
    alloc(&d.bvcnt, nb * 4, "block variance counts");
    alloc(&m->ctr, sizeof(DevCounters), "counters");
    for (int n = 0; n < c.levels; ++n) alloc(&d.vis[n], nb * 16, "visible-block lists");
    for (int n = 0; n < c.levels && n < 2; ++n) alloc(&d.vrect[n], nb * 16, "visible-block lists");
    for (int n = 0; n < c.levels; ++n) {
        const int64_t cap = c.heap_blocks[n] > 0 ? c.heap_blocks[n] : c.max_blocks;
        d.heap_cap[n] = (int32_t)cap;
        const size_t nv = (size_t)cap * (size_t)(side_of(n) * side_of(n) * side_of(n));
        alloc(&d.stack[n], (size_t)cap * 4, "free stack");
        if (n >= 1) alloc(&d.pend[n], (size_t)cap * 4, "pending frees");
        if (n == 0)
            for (int p = 0; p < 2; ++p) alloc(&d.pend0[p], (size_t)cap * 4, "pending frees");
        const size_t pb = (size_t)plane_bytes(c.storage);
        alloc(&d.DW[n], nv * 2 * pb, "TSDF and weight heap");
        alloc(&d.S2[n], nv * pb, "variance heap");
        if (c.color) alloc(&d.C[n], nv * 12, "colour heap");
    }
    m->partials_cap = 2048;
    alloc(&m->partials, (size_t)m->partials_cap * 6 * 8, "reduction partials");
    alloc(&m->pose_out, 6 * 8, "pose gradient");
    alloc(&m->count_dev, 8, "extraction counter");
    alloc(&m->dmd, sizeof(DevMap), "map descriptor");
    d.ctr = global(m->ctr);
    if (st == MRH_OK) st = upload_descriptor(m);
    if (st != MRH_OK) {
        free_all(m);
        delete m;
        return st;
    }
    st = mrh_map_reset(m);
    if (st == MRH_OK) st = check_hip(m, hipStreamSynchronize(m->stream), "create");
    if (st != MRH_OK) {
        free_all(m);
        delete m;
        return st;
    }
    *out = m;
    return MRH_OK;
}

void mrh_map_destroy(mrh_map* map) {
    if (!map) return;
    (void)hipStreamSynchronize(map->stream);
    for (auto& r : map->prof) {
        (void)hipEventDestroy(r.start);
        (void)hipEventDestroy(r.stop);
    }
    for (hipEvent_t e : map->event_pool) (void)hipEventDestroy(e);
    free_all(map);
    delete map;
}

mrh_status mrh_map_reset(mrh_map* map) {
    if (!map) return MRH_ERR_INVALID_ARG;
    map->frames = map->frames_at_sync = 0;
    for (int s = 0; s < 16; ++s) map->stats_at_sync[s] = 0;
    stream_clear(map);
    const uint32_t n_hash = map->dm.hmask + 1;
    launch(map, K_RESET, [&] { hipLaunchKernelGGL(k_reset, dim3(1024), dim3(256), 0, map->stream, map->dmd, n_hash); });
    return check_hip(map, hipGetLastError(), "reset");
}

static void fill_stats(const unsigned long long* s, unsigned long long frames, uint32_t nblocks, uint32_t flags,
                       mrh_stats* out) {
    std::memset(out, 0, sizeof(*out));
    out->frames = (int64_t)frames;
    out->valid_points = (int64_t)s[S_VALID];
    out->dropped_points = (int64_t)s[S_DROPPED];
    out->new_blocks = (int64_t)s[S_NEW];
    out->observations = (int64_t)s[S_OBS];
    for (int n = 0; n < 4; ++n) out->merges[n] = (int64_t)s[S_MERGE0 + n];
    out->failed_inserts = (int64_t)s[S_FAILED];
    out->fresh_observations = (int64_t)s[S_OBS_FRESH];
    out->distinct_voxels = (int64_t)s[S_DISTINCT];
    out->candidate_keys = (int64_t)s[S_CAND];
    out->queued_blocks = (int64_t)s[S_QUEUED];
    out->blocks = (int64_t)nblocks;
    out->error_flags = flags;
}

mrh_status mrh_sync(mrh_map* map, mrh_stats* last, mrh_stats* totals) {
    if (!map) return MRH_ERR_INVALID_ARG;
    DevCounters h;
    mrh_status st = check_hip(map, hipMemcpyAsync(&h, map->ctr, sizeof(h), hipMemcpyDeviceToHost, map->stream), "sync");
    if (st == MRH_OK) st = check_hip(map, hipStreamSynchronize(map->stream), "sync");
    if (st != MRH_OK) return st;
    const uint32_t nb = h.n_blocks < map->dm.max_blocks ? h.n_blocks : map->dm.max_blocks;
    unsigned long long tot[16], since[16];
    for (int s = 0; s < 16; ++s) {
        tot[s] = 0;
        for (int k = 0; k < kStripes; ++k) tot[s] += h.frame[k][s];
        since[s] = tot[s] - map->stats_at_sync[s];
        map->stats_at_sync[s] = tot[s];
    }
    const uint32_t frames_since = map->frames - map->frames_at_sync;
    map->frames_at_sync = map->frames;
    const uint32_t live = nb - (uint32_t)(map->gone < nb ? map->gone : nb);
    if (last) fill_stats(since, frames_since, live, h.error_flags.v, last);
    if (totals) fill_stats(tot, map->frames, live, h.error_flags.v, totals);
    if (h.error_flags.v) {
        const uint32_t zero = 0;
        st = check_hip(map, hipMemcpyAsync(&map->ctr->error_flags.v, &zero, 4, hipMemcpyHostToDevice, map->stream),
                       "clear errors");
        if (st == MRH_OK) st = check_hip(map, hipStreamSynchronize(map->stream), "clear errors");
        if (st != MRH_OK) return st;
        if (h.error_flags.v & kErrTableFull)
            return set_error(map, MRH_ERR_TABLE_FULL, "hash table full (probe limit %d)", map->dm.max_probe);
        if (h.error_flags.v & kErrHeapFull) return set_error(map, MRH_ERR_HEAP_FULL, "a level heap ran out of blocks");
        return set_error(map, MRH_ERR_BLOCK_LIMIT, "more than %u blocks", map->dm.max_blocks);
    }
    return MRH_OK;
}

mrh_status mrh_extract_blocks(mrh_map* map, int32_t* keys_dev, uint8_t* levels_dev, int64_t* offsets_dev,
                              float* D_dev, uint32_t* W_dev, float* S2_dev, int64_t block_cap, int64_t voxel_cap,
                              int64_t* n_blocks, int64_t* n_voxels) {
    if (!map) return MRH_ERR_INVALID_ARG;
    uint32_t nout = 0;
    int64_t nvox = 0;
    mrh_status st = scan_rows(map, "extract", nout, nvox);
    if (st != MRH_OK) return st;
    if (n_blocks) *n_blocks = nout;
    if (n_voxels) *n_voxels = nvox;
    const bool want_blocks = keys_dev || levels_dev || offsets_dev;
    const bool want_vox = D_dev || W_dev || S2_dev;
    if (!want_blocks && !want_vox) return MRH_OK;
    if (block_cap < (int64_t)nout || (want_vox && voxel_cap < nvox))
        return set_error(map, MRH_ERR_BUFFER_TOO_SMALL, "extract needs %u blocks / %lld voxels", nout, (long long)nvox);
    if (nout == 0) {
        if (offsets_dev) return check_hip(map, hipMemcpy(offsets_dev, &nvox, 8, hipMemcpyHostToDevice), "extract");
        return MRH_OK;
    }
    const dim3 grid(extract_grid(nout));
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, map->stream, map->dmd, map->extract_rows, nout, keys_dev, levels_dev,
                           offsets_dev, D_dev, W_dev, S2_dev);
    };
    switch (map->cfg.storage) {
        case MRH_STORE_F16: run(k_extract<MRH_STORE_F16>); break;
        case MRH_STORE_BF16: run(k_extract<MRH_STORE_BF16>); break;
        default: run(k_extract<MRH_STORE_F32>);
    }
    st = check_hip(map, hipGetLastError(), "extract");
    if (st == MRH_OK) st = check_hip(map, hipStreamSynchronize(map->stream), "extract");
    return st;
}

mrh_status mrh_profile_enable(mrh_map* map, int32_t on) {
    if (!map) return MRH_ERR_INVALID_ARG;
    map->profiling = on != 0;
    return MRH_OK;
}

mrh_status mrh_profile_collect(mrh_map* map, double* ms, int64_t* launches, int32_t n_kernels) {
    if (!map || n_kernels < 0 || (n_kernels > 0 && (!ms || !launches))) return MRH_ERR_INVALID_ARG;
    mrh_status st = check_hip(map, hipStreamSynchronize(map->stream), "profile");
    if (st != MRH_OK) return st;
    for (int k = 0; k < n_kernels; ++k) ms[k] = 0.0, launches[k] = 0;
    for (auto& r : map->prof) {
        float t = 0.f;
        if (hipEventElapsedTime(&t, r.start, r.stop) == hipSuccess && r.kernel < n_kernels) {
            ms[r.kernel] += (double)t;
            launches[r.kernel] += 1;
        }
        map->event_pool.push_back(r.start);
        map->event_pool.push_back(r.stop);
    }
    map->prof.clear();
    return MRH_OK;
}

}  // extern "C"

namespace mrh {
hipEvent_t take_event(mrh_map* m) {
    if (!m->event_pool.empty()) {
        hipEvent_t e = m->event_pool.back();
        m->event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    return e;
}

}  // namespace mrh
