// LiDAR fusion work units (Sec. 3.1 "3D Point Cloud", Eq. 1; Eq. 3 and Eq. 5; Sec. 3.2.1),
// shared by the single-map kernels (points.hip) and the batched kernels (batch.hip).
//
//   points_alloc_chunk  4 to 16 rays: validity, segment [o, p + tau n] (carving) or the band
//                       [p - tau n, p + tau n], walk over the block lattice,
//                       insert, and the record of the hash slots of each ray's blocks in walk order
//   points_ray_chunk    4 to 16 rays: their recorded (ray, block) pairs in parallel; inside each block a
//                       walk over the block's own voxel lattice; each crossed voxel gets
//                       clip((p - x) . n, -tau, tau).
//                       Saturated observations (+tau) only bump an integer count; the others add
//                       their fixed-point value q = rint(d 2^24) and its square q^2 to exact integer
//                       sums, so the accumulation is order-independent and needs no read of the
//                       voxel's state; the update forms the sums of (d - D) and (d - D)^2 from them.
//                       The touched lane groups of each block are marked
//   queue_touched       the touched blocks onto their levels' update queues
//   points_update_task  8 queued blocks of level 0, 1 or 2, or 64 of level 3, per wave: each voxel's
//                       scan statistics merge into its state (W' = W + n, D' = D + s1 / W',
//                       S2' = S2 + s2 - s1^2 / W', the batch form of Eq. 3 and Eq. 5), then the
//                       block variance bookkeeping and the merging criterion
#pragma once

#include "mrh_update.h"

namespace mrh {

constexpr double kS1Scale = 16777216.0;         // 2^24 per metre: q = rint(d 2^24), |q| <= tau 2^24
constexpr double kS2Scale = 281474976710656.0;  // 2^48 per square metre: the sum of q^2

struct ScanParams {
    int32_t parity;  // the frame's parity (selects the double-buffered per-frame counts)
    int32_t rays;    // rays per workgroup (at most kGroupRays)
    Pose P;
    const float MRH_GLOBAL* xyz;  // device points, sensor frame, [n][3]
    int64_t n;
};

__device__ inline bool point_segment(const DevMap& m, const ScanParams& sp, int64_t i, double a[3], double e[3],
                                     double p[3], double n[3]) {
    const float MRH_GLOBAL* __restrict__ xyz = sp.xyz;
    const double ps[3] = {(double)xyz[3 * i], (double)xyz[3 * i + 1], (double)xyz[3 * i + 2]};
    if (!(__builtin_isfinite(ps[0]) && __builtin_isfinite(ps[1]) && __builtin_isfinite(ps[2]))) return false;
    const double r2 = (ps[0] * ps[0] + ps[1] * ps[1]) + ps[2] * ps[2];
    if (!(r2 >= m.r2lo && r2 <= m.r2hi)) return false;
    pose_apply(sp.P, ps, p);
    unit_direction(p, sp.P.t, n);
    for (int k = 0; k < 3; ++k) {
        a[k] = m.carve ? sp.P.t[k] : p[k] - m.tau * n[k];
        e[k] = p[k] + m.tau * n[k];
    }
    return true;
}

// One axis of a ray's block walk (the walk's lattice has the blocks as cells): the parameter of its i-th
// boundary is ((c + s i + (s > 0)) - A) iD, evaluated as Walk does.
struct RayAxis {
    double A, iD;
    double reach;      // cells the segment spans, |E - A|
    double to_first;   // distance to the first boundary, in cells
    int32_t c, s, n;   // first cell, direction, boundaries crossed (parameter <= 1)

    __device__ inline void init(double a, double e, double inv_cell) {
        int32_t guard = 0;
        double t;
        int st;
        walk_axis(a, e, inv_cell, A, c, st, iD, t, guard);
        s = st;
        const double b0 = (double)(c + (s > 0 ? 1 : 0));
        reach = __builtin_fabs(e * inv_cell - A);
        to_first = s > 0 ? b0 - A : A - b0;
        // the cells between the segment's ends; the last boundary may round to either side of its end
        n = s == 0 ? 0 : guard;
        if (n > 0 && !(at(n - 1) <= 1.0)) --n;
        if (s != 0 && at(n) <= 1.0) ++n;
    }
    __device__ inline double at(int32_t i) const { return ((double)(c + s * i + (s > 0 ? 1 : 0)) - A) * iD; }
    // Boundaries with a parameter below t (at_most: not above t).  The parameters do not decrease with i
    // (a rounded difference times a constant), and the estimate is off by one at most (its rounding errors
    // stay far below a cell).
    __device__ inline int32_t before(double t, bool at_most) const {
        const double m = __builtin_floor(t * reach - to_first) + 1.0;
        int32_t k = m < 0.0 ? 0 : m < (double)n ? (int32_t)m : n;
        const double lo = at(k - 1), hi = at(k);
        if (k > 0 && !(at_most ? lo <= t : lo < t)) return k - 1;
        return k + (k < n && (at_most ? hi <= t : hi < t) ? 1 : 0);
    }
};

// The ray j of a workgroup's kGroupRays with first[j] <= q < first[j + 1] (prefix sums in LDS).
constexpr int kGroupRays = 16;

__device__ inline int ray_of(const uint32_t* first, uint32_t q) {
    int j = 0;
#pragma unroll
    for (int step = kGroupRays / 2; step > 0; step >>= 1)
        if (q >= first[j + step]) j += step;
    return j;
}

// Rays per 256-thread workgroup of the allocation launch, and the blocks it takes at a time.
constexpr int kAllocRaysPerGroup = kGroupRays;
constexpr int kAllocUnroll = 2;
constexpr int kAllocRound = 256 * kAllocUnroll;
constexpr int kAllocNew = 512;  // new blocks a workgroup registers together

// Allocation for rays chunk * sp.rays ..: the blocks of each ray's walk, their
// insert, and the record of the hash slots of each ray's blocks in walk order.  The walk
// takes the boundaries of the three axes in the order of their parameters, lowest axis on ties, so the
// place of a boundary in it is its index plus the boundaries of the other two axes before it, and the
// block behind it follows from the same counts: every block is found on its own, one thread per block,
// with no chain along the ray.  Walked step by step, a launch took as long as its longest ray, about
// 250 blocks, whatever the number of rays: first, second and a later scan of 8000 points in a room 197, 92 and
// 90 us, so 117, 15 and 11; of 131072 points 493, 131 and 131 us, so 272, 61 and 55.
__device__ inline void points_alloc_chunk(const DevMap& m, const ScanParams& sp, uint32_t chunk) {
    __shared__ RayAxis axes[kAllocRaysPerGroup][3];
    __shared__ uint32_t sfirst[kAllocRaysPerGroup + 1];
    // the keys the workgroup inserted, registered at its end with one allocation atomic
    __shared__ unsigned long long nkey[kAllocNew], nold;
    __shared__ uint32_t nslot[kAllocNew], ncount;
    const int lane = lane_id(), tid = (int)threadIdx.x;
    const int64_t r0 = (int64_t)chunk * sp.rays;
    if (tid < 64) {
        const int64_t i = r0 + lane;
        const bool mine = lane < sp.rays && i < sp.n;
        double a[3], e[3], p[3], nn[3];
        const bool ok = mine && point_segment(m, sp, i, a, e, p, nn);
        const unsigned long long vmask = __ballot(ok);
        const bool in_range = ok && segment_in_range(a, e, m.invB);
        const unsigned long long dmask = __ballot(ok && !in_range);
        uint32_t cnt = 0;
        if (in_range) {
            cnt = 1;
            for (int k = 0; k < 3; ++k) {
                RayAxis x;
                x.init(a[k], e[k], m.invB);
                axes[lane][k] = x;
                cnt += (uint32_t)x.n;
            }
        }
        if (mine) m.rcount[i] = cnt;
        uint32_t incl = cnt;
        for (int o = 1; o < kAllocRaysPerGroup; o <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)incl, o);
            if (lane >= o) incl += v;
        }
        if (lane < kAllocRaysPerGroup) sfirst[lane + 1] = incl;
        if (lane == kAllocRaysPerGroup - 1) stat_add(m, S_CAND, (unsigned long long)incl);
        if (lane == 0) {
            sfirst[0] = ncount = 0u;
            stat_add(m, S_VALID, (unsigned long long)__popcll(vmask));
            stat_add(m, S_DROPPED, (unsigned long long)__popcll(dmask));
        }
    }
    __syncthreads();
    // blocks [sfirst[j], sfirst[j + 1]) are ray j's: its first block, then those behind the boundaries of
    // axis 0, 1 and 2
    const uint32_t total = sfirst[kAllocRaysPerGroup], K = (uint32_t)m.rcap_k;
    for (uint32_t base = (uint32_t)(tid & ~63); base < total; base += kAllocRound) {  // wave-uniform
        unsigned long long key[kAllocUnroll], seen[kAllocUnroll];
        uint32_t slot[kAllocUnroll], place[kAllocUnroll];
        int ray[kAllocUnroll];
        uint32_t open = 0, absent = 0;  // bits u: still probing / met an empty slot
#pragma unroll
        for (int u = 0; u < kAllocUnroll; ++u) {
            const uint32_t q = base + 256u * u + (uint32_t)lane;
            key[u] = seen[u] = kEmptyKey;
            slot[u] = kInvalidId;
            place[u] = 0;
            ray[u] = 0;
            if (q >= total) continue;
            ray[u] = ray_of(sfirst, q);
            const uint32_t f = sfirst[ray[u]];
            const RayAxis* x = axes[ray[u]];
            int32_t i = (int32_t)(q - f) - 1;
            int32_t n0 = 0, n1 = 0, n2 = 0;  // boundaries of each axis behind the block
            if (i >= 0) {
                const int32_t x0 = x[0].n, x1 = x[1].n;
                const int k = i < x0 ? 0 : i < x0 + x1 ? 1 : 2;
                if (k >= 1) i -= x0;
                if (k == 2) i -= x1;
                const double t = x[k].at(i);
                n0 = k == 0 ? i + 1 : x[0].before(t, true);
                n1 = k == 1 ? i + 1 : x[1].before(t, k > 1);
                n2 = k == 2 ? i + 1 : x[2].before(t, false);
            }
            place[u] = (uint32_t)(n0 + n1 + n2);
            const int32_t c0 = x[0].c + x[0].s * n0, c1 = x[1].c + x[1].s * n1, c2 = x[2].c + x[2].s * n2;
            key[u] = pack_key(c0, c1, c2);
            slot[u] = spatial_hash(c0, c1, c2) & m.hmask;
            open |= 1u << u;
        }
        const uint32_t valid = open;
        // probe through the caches: a key found there is in the table (keys never leave it while a launch
        // inserts), and one that seems absent is looked up again past the caches below
        for (int p = 0; __ballot(open != 0); ++p) {
#pragma unroll
            for (int u = 0; u < kAllocUnroll; ++u)
                if ((open >> u) & 1u) seen[u] = m.table[slot[u]].key;
#pragma unroll
            for (int u = 0; u < kAllocUnroll; ++u) {
                if (!((open >> u) & 1u)) continue;
                if (seen[u] == key[u]) {
                    open &= ~(1u << u);
                } else if (seen[u] == kEmptyKey || p + 1 >= m.max_probe) {
                    open &= ~(1u << u);
                    absent |= 1u << u;
                } else {
                    slot[u] = (slot[u] + 1) & m.hmask;
                }
            }
        }
        // insert what was absent, from the empty slot met: a read past the caches first (most absent keys
        // have been inserted by another ray meanwhile), then the CAS; all of a step in flight together
        uint32_t fresh = 0;  // bits u: this lane inserted key[u]
        open = absent;
        while (__ballot(open != 0)) {
#pragma unroll
            for (int u = 0; u < kAllocUnroll; ++u)
                if ((open >> u) & 1u)
                    seen[u] = __hip_atomic_load(&m.table[slot[u]].key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int u = 0; u < kAllocUnroll; ++u)
                if (((open >> u) & 1u) && seen[u] == kEmptyKey) {
                    seen[u] = atomicCAS(&m.table[slot[u]].key, kEmptyKey, key[u]);
                    if (seen[u] == kEmptyKey) fresh |= 1u << u, seen[u] = key[u];
                }
#pragma unroll
            for (int u = 0; u < kAllocUnroll; ++u) {
                if (!((open >> u) & 1u)) continue;
                if (seen[u] == key[u]) {
                    open &= ~(1u << u);
                } else if (((slot[u] - home_slot(key[u], m.hmask)) & m.hmask) + 1u >= (uint32_t)m.max_probe) {
                    open &= ~(1u << u);
                    slot[u] = kInvalidId;
                    atomicOr(&m.ctr->error_flags.v, kErrTableFull);
                } else {
                    slot[u] = (slot[u] + 1) & m.hmask;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kAllocUnroll; ++u) {
            const bool is_new = (fresh >> u) & 1u;
            const unsigned long long mask = __ballot(is_new);
            if (!mask) continue;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&ncount, (uint32_t)__popcll(mask));
            at = uniform(at) + (uint32_t)rank_in_mask(mask);
            const bool spill = is_new && at >= (uint32_t)kAllocNew;
            if (is_new && !spill) nkey[at] = key[u], nslot[at] = slot[u];
            register_new(m, spill, key[u], slot[u]);
        }
#pragma unroll
        for (int u = 0; u < kAllocUnroll; ++u) {
            if (((valid >> u) & 1u) && place[u] < K) m.rslots[(size_t)(r0 + ray[u]) * K + place[u]] = slot[u];
            // a key that lanes of the wave ask for together is one lost insert
            unsigned long long left = __ballot(((valid >> u) & 1u) && slot[u] == kInvalidId);
            while (left) {
                left &= ~__ballot(key[u] == shfl_u64(key[u], __ffsll((long long)left) - 1));
                if (lane == 0) stat_add(m, S_FAILED, 1ull);
            }
        }
    }
    __syncthreads();
    const uint32_t nnew = ncount < (uint32_t)kAllocNew ? ncount : (uint32_t)kAllocNew;
    if (nnew == 0) return;
    if (tid == 0) nold = take_new_blocks(m, nnew);
    __syncthreads();
    for (uint32_t i = (uint32_t)tid; i < nnew; i += 256)
        register_block(m, nkey[i], nslot[i], (uint32_t)nold + i, (uint32_t)(nold >> 32) + i);
}

// Saturated (+tau) observations are counted in a workgroup-private LDS table first where the
// workgroup's rays, neighbours in azimuth, tend to cross the same voxels: in blocks of level 1 to 3, and
// in finest ones near the sensor (every ray of a scan starts there).  The table is flushed with one
// global atomic per distinct voxel once the rays are done.  The counts are integers, so the result
// equals adding them one at a time.  An entry is (key + 1) << 32 | count with key = level << 30 |
// heap position; keys are never removed while rays run.
constexpr int kSatBits = 11;
constexpr int kSatSlots = 1 << kSatBits;
constexpr double kSatNear = 100.0;  // level-0 blocks whose centre is within 100 voxel edges of the origin use it

struct SatTable {
    unsigned long long e[kSatSlots];
};

__device__ inline void sat_table_clear(SatTable& tab) {
    for (int k = threadIdx.x; k < kSatSlots; k += blockDim.x) tab.e[k] = 0ull;
    __syncthreads();
}

// Count one saturated observation in the table: 0 when the voxel must go to global memory (heap
// position too large for a key, or no free entry within 4 probes), 2 when it is the voxel's first there.
__device__ inline int sat_table_add(SatTable& tab, int level, size_t at) {
    if (at >= (size_t)((1u << 30) - 1u)) return 0;
    const uint32_t key = (((uint32_t)level << 30) | (uint32_t)at) + 1u;
    uint32_t h = (key * 2654435761u) >> (32 - kSatBits);
    for (int p = 0; p < 4; ++p) {
        uint32_t k = (uint32_t)(__hip_atomic_load(&tab.e[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >> 32);
        if (k == 0u) {
            k = (uint32_t)(atomicCAS(&tab.e[h], 0ull, ((unsigned long long)key << 32) | 1ull) >> 32);
            if (k == 0u) return 2;
        }
        if (k == key) {
            atomicAdd(&tab.e[h], 1ull);
            return 1;
        }
        h = (h + 1) & (kSatSlots - 1);
    }
    return 0;
}

// Mark lane groups of block `id` as touched: most rays through a block find their groups already
// marked, so reading first keeps the same-address atomics off the memory side.
__device__ inline void touch_block(const DevMap& m, uint32_t id, unsigned long long groups) {
    if ((m.btouch[id] & groups) != groups) atomicOr(&m.btouch[id], groups);
}

// All threads of the workgroup: add the table's counts to the global accumulators.
__device__ inline void sat_table_flush(const DevMap& m, SatTable& tab) {
    __syncthreads();
    for (int k = threadIdx.x; k < kSatSlots; k += blockDim.x) {
        const unsigned long long e = tab.e[k];
        if (e) {
            const uint32_t code = (uint32_t)(e >> 32) - 1u;
            atomicAdd(of_level(m.acc_sat, (int)(code >> 30)) + (code & ((1u << 30) - 1u)), (uint32_t)e);
        }
    }
}

// A band observation d of a block's voxel `at`: 1, q and q^2 (q its fixed-point
// value) are added, exact integers, fire-and-forget atomics with no dependent load.  The count rides on
// the sum of q, made non-negative by band_bias: two atomics per observation instead of three (band
// observations were two thirds of a scan's atomics).  A scan whose sums could outgrow the shared
// word (m.band_wide) keeps the count in a word of its own, and one whose squares could outgrow theirs
// (m.square_wide) the halves of each square in two: scans of such a map run the WIDE kernels (with that test
// in the common ones a pass of three scans of 31 x 1023 rays, with its extraction, took 3.96 -> 4.07 ms).
constexpr int kBandShift = 44;  // count << 44 | sum of q + bias

// Where a block's words are (count: where it is kept apart, else null): from word `base` of its level.
struct BandAcc {
    unsigned long long MRH_GLOBAL* s1;
    unsigned long long MRH_GLOBAL* s2;
    uint32_t MRH_GLOBAL* count;
    int level;
    size_t base;
};

template <bool WIDE>
__device__ inline void accumulate_band(const DevMap& m, const BandAcc& a, uint32_t at, double d) {
    const long long q = (long long)__builtin_rint(d * kS1Scale);
    if (a.count) {
        atomicAdd(a.count + at, 1u);
        atomicAdd(a.s1 + at, (unsigned long long)q);
    } else {
        atomicAdd(a.s1 + at, (1ull << kBandShift) + (unsigned long long)(q + m.band_bias));
    }
    if (WIDE && m.square_wide) {
        const unsigned long long u = (unsigned long long)(q < 0 ? -q : q), low = u * u;
        atomicAdd(a.s2 + at, low & 0xFFFFFFFFull);
        atomicAdd(of_level(m.acc_s2h, a.level) + a.base + at, __umul64hi(u, u) << 32 | low >> 32);
    } else {
        atomicAdd(a.s2 + at, (unsigned long long)(q * q));
    }
}

// The count and the sum of q of a voxel from its words.
__device__ inline void band_sums(const DevMap& m, uint32_t wide_count, unsigned long long word, uint32_t& n,
                                 unsigned long long& s1) {
    if (m.band_wide) {
        n = wide_count;
        s1 = word;
    } else {
        n = (uint32_t)(word >> kBandShift);
        s1 = (word & ((1ull << kBandShift) - 1ull)) - (unsigned long long)n * (unsigned long long)m.band_bias;
    }
}

// The sum of a voxel's squares, in square metres: `low` is its word of acc_s2, and the other word is read
// and left at zero.
template <bool WIDE>
__device__ inline double take_squares(const DevMap& m, int level, size_t at, unsigned long long low) {
    if (!WIDE || !m.square_wide) return (double)low / kS2Scale;
    const unsigned long long high = m.acc_s2h[level][at] + (low >> 32);
    m.acc_s2h[level][at] = 0ull;
    low &= 0xFFFFFFFFull;
    return (high >> 32 ? (double)high * 0x1p32 + (double)low : (double)(high << 32 | low)) / kS2Scale;
}

// The block walk restricted to one block: the segment is clipped to the block's box, the walk
// starts in the (clamped) cell of the clipped entry point and steps on the block's own lattice of
// side^3 voxels until it leaves the block or passes the clipped exit parameter.
struct BoxWalk {
    double A0, A1, A2, iD0, iD1, iD2, t0, t1, t2, tout;
    int c0, c1, c2, s0, s1, s2, side;

    __device__ static inline void axis(double a, double e, double ob, double inv_nu, int side, double& A, double& D,
                                       double& iD, int& st, double& tin, double& tout) {
        A = (a - ob) * inv_nu;
        const double El = (e - ob) * inv_nu;
        D = El - A;
        if (D != 0.0) {
            iD = 1.0 / D;
            const double nearb = D > 0.0 ? 0.0 : (double)side;
            const double farb = D > 0.0 ? (double)side : 0.0;
            const double ta = (nearb - A) * iD;
            const double tb = (farb - A) * iD;
            if (ta > tin) tin = ta;
            if (tb < tout) tout = tb;
            st = D > 0.0 ? 1 : -1;
        } else {
            iD = 0.0;
            st = 0;
        }
    }
    __device__ static inline void start(double A, double D, double iD, int st, double tin, int side, int& c, double& t) {
        double fl = __builtin_floor(A + tin * D);
        if (fl < 0.0) fl = 0.0;
        if (fl > (double)(side - 1)) fl = (double)(side - 1);
        c = (int)fl;
        t = st != 0 ? ((double)(c + (st > 0 ? 1 : 0)) - A) * iD : __builtin_inf();
    }
    __device__ inline void init(const double a[3], const double e[3], const int32_t b[3], double B, double inv_nu,
                                int side_) {
        side = side_;
        double D0, D1, D2, tin = 0.0;
        tout = 1.0;
        axis(a[0], e[0], (double)b[0] * B, inv_nu, side, A0, D0, iD0, s0, tin, tout);
        axis(a[1], e[1], (double)b[1] * B, inv_nu, side, A1, D1, iD1, s1, tin, tout);
        axis(a[2], e[2], (double)b[2] * B, inv_nu, side, A2, D2, iD2, s2, tin, tout);
        start(A0, D0, iD0, s0, tin, side, c0, t0);
        start(A1, D1, iD1, s1, tin, side, c1, t1);
        start(A2, D2, iD2, s2, tin, side, c2, t2);
    }
    // step to the next voxel; the axis stepped along, or -1 once the walk left the block
    __device__ inline int next() {
        double tm = t0;
        int k = 0;
        if (t1 < tm) tm = t1, k = 1;
        if (t2 < tm) tm = t2, k = 2;
        if (!(tm <= tout)) return -1;
        if (k == 0) {
            c0 += s0;
            if (c0 < 0 || c0 >= side) return -1;
            t0 = ((double)(c0 + (s0 > 0 ? 1 : 0)) - A0) * iD0;
        } else if (k == 1) {
            c1 += s1;
            if (c1 < 0 || c1 >= side) return -1;
            t1 = ((double)(c1 + (s1 > 0 ? 1 : 0)) - A1) * iD1;
        } else {
            c2 += s2;
            if (c2 < 0 || c2 >= side) return -1;
            t2 = ((double)(c2 + (s2 > 0 ? 1 : 0)) - A2) * iD2;
        }
        return k;
    }
};

// A ray's part of the launch: segment a..e, surface point p, direction n.
struct RaySegment {
    double a[3], e[3], p[3], n[3];
};

// The blocks the scan's rays touched (non-zero touch mask), queued per level for the update: block
// ids first .. first + count - 1 of this workgroup's range, positions taken in LDS and one atomic
// per level per workgroup (every thread of the workgroup calls).
constexpr int kTouchPerThread = 8;

__device__ inline void queue_touched(const DevMap& m, uint32_t first, uint32_t count, int par) {
    __shared__ uint32_t lcnt[4], lbase[4];
    if (threadIdx.x < 4) lcnt[threadIdx.x] = 0;
    __syncthreads();
    int lvl[kTouchPerThread];
    uint32_t pos[kTouchPerThread];
    for (int r = 0; r < kTouchPerThread; ++r) {
        const uint32_t k = (uint32_t)r * blockDim.x + threadIdx.x;  // consecutive threads, consecutive ids
        lvl[r] = -1;
        pos[r] = 0;
        if (k < count && m.btouch[first + k] != 0ull) {
            lvl[r] = (int)((m.binfo[first + k] >> kLevelShift) & 3u);
            pos[r] = atomicAdd(&lcnt[lvl[r]], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < 4 && lcnt[threadIdx.x]) lbase[threadIdx.x] = atomicAdd(&m.ctr->vis_n[par][threadIdx.x].v, lcnt[threadIdx.x]);
    __syncthreads();
    for (int r = 0; r < kTouchPerThread; ++r) {
        if (lvl[r] < 0) continue;
        const uint32_t id = first + (uint32_t)r * blockDim.x + threadIdx.x;
        m.vis[lvl[r]][lbase[lvl[r]] + pos[r]] = make_entry(id, m.binfo[id], m.bkey[id]);
    }
}

// The lane groups that the workgroup's rays touched in blocks of level 0 .. 2, per block id, until
// the rays are done.
constexpr int kTouchBits = 9;
constexpr int kTouchSlots = 1 << kTouchBits;

struct TouchTable {
    unsigned long long groups[kTouchSlots];
    uint32_t id[kTouchSlots];  // block id + 1, 0 empty
};

__device__ inline void touch_table_clear(TouchTable& t) {
    for (int k = threadIdx.x; k < kTouchSlots; k += blockDim.x) t.groups[k] = 0ull, t.id[k] = 0u;
}

__device__ inline void touch_table_add(const DevMap& m, TouchTable& t, uint32_t id, unsigned long long groups) {
    uint32_t h = (id * 2654435761u) >> (32 - kTouchBits);
    for (int p = 0; p < 8; ++p) {
        const uint32_t old = atomicCAS(&t.id[h], 0u, id + 1u);
        if (old == 0u || old == id + 1u) {
            atomicOr(&t.groups[h], groups);
            return;
        }
        h = (h + 1) & (kTouchSlots - 1);
    }
    touch_block(m, id, groups);
}

__device__ inline void touch_table_flush(const DevMap& m, const TouchTable& t) {
    for (int k = threadIdx.x; k < kTouchSlots; k += blockDim.x)
        if (t.id[k]) touch_block(m, t.id[k] - 1u, t.groups[k]);
}

// Rays per 256-thread workgroup of the ray launch at most, and the pairs it takes at a time.
constexpr int kRaysPerGroup = kGroupRays;
constexpr int kRayUnroll = 3;
constexpr int kRayRound = 256 * kRayUnroll;

struct RayLds {
    SatTable tab;
    TouchTable touch;
    RaySegment seg[kRaysPerGroup];
    u32x4 pair[kRayRound];      // the round's pairs: hash slot (key, block id, row)
    uint8_t ray[kRayRound];     // and ray
    uint16_t wait[kRayRound];   // waiting pairs
    uint32_t first[kRaysPerGroup + 1];
    uint32_t n[2];              // waiting pairs of level 0 (from the front) / of levels 1 and 2 (from the back)
};
// the serial walks past the recorded blocks wait behind the pairs of a round that has 256 at most
static_assert(sizeof(Walk) * kRaysPerGroup <= sizeof(u32x4) * (kRayRound - 256), "room for the walks");

// The ray's one observation in a level-3 block: the centre of its only voxel (Eq. 1).
template <bool WIDE>
__device__ inline void ray_coarse_block(const DevMap& m, const RaySegment& r, const HashSlot& hs, RayLds& L) {
    int32_t b[3];
    unpack_key(hs.key, b[0], b[1], b[2]);
    double t[3];
    for (int k = 0; k < 3; ++k) t[k] = (r.p[k] - ((double)b[k] * m.B + 0.5 * m.nu[3])) * r.n[k];
    const double sd = (t[0] + t[1]) + t[2];
    const double d = sd < -m.tau ? -m.tau : (sd > m.tau ? m.tau : sd);
    const size_t at = (size_t)(hs.info & kSlotMask);
    int counted = 0;
    if (d >= m.tau) {
        counted = sat_table_add(L.tab, 3, at);
        if (!counted) atomicAdd(&m.acc_sat[3][at], 1u);
    } else {
        accumulate_band<WIDE>(m, BandAcc{m.acc_s1[3] + at, m.acc_s2[3] + at, m.band_wide ? m.acc_band[3] + at : nullptr, 3, at}, 0u, d);
    }
    if (counted != 1) touch_table_add(m, L.touch, hs.id, 1ull);  // (1: marked with the voxel's first)
}

// The observations of one ray inside a block of level 0 .. 2 (slot and level in `info`): the block walk
// restricted to the block's own voxel lattice.  The terms of Eq. 1's product are kept per axis and
// re-evaluated (the whole expression) on the axis that stepped.
template <bool WIDE>
__device__ inline void ray_fine_block(const DevMap& m, const double o[3], const RaySegment& r, unsigned long long key,
                                      uint32_t id, uint32_t info, RayLds& L) {
    int32_t b[3];
    unpack_key(key, b[0], b[1], b[2]);
    const int level = (int)((info >> kLevelShift) & 3u), side = 8 >> level;
    const size_t base = (size_t)(info & kSlotMask) << (3 * (3 - level));
    const double nu = nu_of(m.nu, level);
    uint32_t MRH_GLOBAL* const sat = of_level(m.acc_sat, level) + base;
    const BandAcc acc{of_level(m.acc_s1, level) + base, of_level(m.acc_s2, level) + base,
                      m.band_wide ? of_level(m.acc_band, level) + base : nullptr, level, base};
    BoxWalk bw;
    bw.init(r.a, r.e, b, m.B, inv_nu_of(m.inv_nu, level), side);
    const double ob[3] = {(double)b[0] * m.B, (double)b[1] * m.B, (double)b[2] * m.B};
    bool shared = level > 0;
    if (!shared) {
        const double h = 0.5 * m.B, lim = kSatNear * nu;
        const double r0 = ob[0] + h - o[0], r1 = ob[1] + h - o[1], r2 = ob[2] + h - o[2];
        shared = r0 * r0 + r1 * r1 + r2 * r2 < lim * lim;
    }
    auto term = [&](int k, int c) { return (r.p[k] - (ob[k] + ((double)c + 0.5) * nu)) * r.n[k]; };
    double t0 = term(0, bw.c0), t1 = term(1, bw.c1), t2 = term(2, bw.c2);
    unsigned long long groups = 0ull;  // the update's lane groups this ray touches in the block
    for (int s = 0;; ++s) {
        const double sd = (t0 + t1) + t2;
        const double d = sd < -m.tau ? -m.tau : (sd > m.tau ? m.tau : sd);
        const uint32_t mo = (uint32_t)(spread3(bw.c0) | (spread3(bw.c1) << 1) | (spread3(bw.c2) << 2));
        groups |= 1ull << (level == 0 ? mo >> 3 : (level == 1 ? mo : 0u));
        if (d >= m.tau) {
            if (!(shared && sat_table_add(L.tab, level, base + (size_t)mo))) atomicAdd(sat + mo, 1u);
        } else {
            accumulate_band<WIDE>(m, acc, mo, d);
        }
        if (s == 3 * side) break;
        const int k = bw.next();
        if (k < 0) break;
        if (k == 0) t0 = term(0, bw.c0);
        else if (k == 1) t1 = term(1, bw.c1);
        else t2 = term(2, bw.c2);
    }
    touch_table_add(m, L.touch, id, groups);
}

// Traversal and accumulation for rays chunk * sp.rays .. (all threads of the workgroup).  A
// ray's block walk is a serial chain of lookups, so the (ray, block) pairs that the allocation launch
// recorded are processed in parallel instead, kRayRound at a time by the whole workgroup, in two
// steps.  First each thread reads the hash slots of its pairs, all reads of a step together; a pair in a
// level-3 block is one observation, counted at once, and the others wait in LDS, level 0 from the
// front and levels 1 and 2 from the back.  Then full waves of waiting pairs of like length walk their
// blocks.  Reads and atomics are kept apart because a wave's memory operations complete in order: a
// read issued behind the walk's atomics, performed beyond the L2, waits for them (which is also why
// the touched groups are gathered in LDS).  First, second and a later scan of 131072 points in a room:
// 1495, 891 and 270 us by the walk of each ray, so 1050, 496 and 145 (the first has 27 M atomics, and their
// rate, about 25 G/s, bounds it).
// The blocks of a ray beyond the recorded rcap_k are walked afterwards by one thread per ray, through
// the same two steps.
template <bool WIDE>
__device__ inline void points_ray_chunk(const DevMap& m, const ScanParams& sp, uint32_t chunk, RayLds& L) {
    const int lane = lane_id(), tid = (int)threadIdx.x, wv = (int)uniform(threadIdx.x >> 6);
    const int64_t r0 = (int64_t)chunk * sp.rays;
    const uint32_t K = (uint32_t)m.rcap_k;
    const uint32_t cnt = (tid < sp.rays && r0 + tid < sp.n) ? m.rcount[r0 + tid] : 0u;
    if (cnt > 0) {
        RaySegment s;
        point_segment(m, sp, r0 + tid, s.a, s.e, s.p, s.n);  // valid: the ray has recorded blocks
        L.seg[tid] = s;
    }
    if (wv == 0) {
        const uint32_t c = cnt < K ? cnt : K;
        uint32_t incl = c;
        for (int o = 1; o < kRaysPerGroup; o <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)incl, o);
            if (lane >= o) incl += v;
        }
        if (lane < kRaysPerGroup) L.first[lane + 1] = incl;
        if (lane == 0) L.first[0] = 0u;
    }
    touch_table_clear(L.touch);
    sat_table_clear(L.tab);  // (ends with a barrier)
    // pairs [first[j], first[j + 1]) are ray j's
    const uint32_t total = L.first[kRaysPerGroup];
    bool more = cnt > K;     // this thread's ray has unrecorded blocks
    bool tail = false;       // their walks have begun
    for (uint32_t base = 0;;) {
        const bool recorded = base < total;
        if (!recorded && !__syncthreads_or(more ? 1 : 0)) break;
        if (tid < 2) L.n[tid] = 0u;
        __syncthreads();
        if (recorded) {
            uint32_t slot[kRayUnroll];
            u32x4 hs[kRayUnroll];
#pragma unroll
            for (int u = 0; u < kRayUnroll; ++u) {
                const uint32_t q = base + 256u * u + (uint32_t)tid;
                slot[u] = kInvalidId;
                if (q < total) {
                    const int j = ray_of(L.first, q);
                    L.ray[256 * u + tid] = (uint8_t)j;
                    slot[u] = m.rslots[(size_t)(r0 + j) * K + (q - L.first[j])];
                }
            }
#pragma unroll
            for (int u = 0; u < kRayUnroll; ++u) {
                hs[u] = u32x4{0u, 0u, kInvalidId, kNoBlockBit};
                if (slot[u] != kInvalidId) hs[u] = load_as<u32x4>(m.table + slot[u]);
            }
#pragma unroll
            for (int u = 0; u < kRayUnroll; ++u) L.pair[256 * u + tid] = hs[u];
            base += kRayRound;
        } else {
            // one block per ray and round
            HashSlot hs{0ull, kInvalidId, kNoBlockBit};
            L.ray[tid] = (uint8_t)(tid & (kRaysPerGroup - 1));
            Walk* walk = reinterpret_cast<Walk*>(L.pair + 256);
            if (more) {
                Walk w;
                if (tail) {
                    w = walk[tid];
                } else {
                    w.init(L.seg[tid].a, L.seg[tid].e, m.invB);
                    for (uint32_t s = 0; s < K; ++s) w.next();
                }
                hs = find_slot(m, pack_key(w.c0, w.c1, w.c2));
                more = w.next();
                walk[tid] = w;
            }
            L.pair[tid] = u32x4{(uint32_t)hs.key, (uint32_t)(hs.key >> 32), hs.id, hs.info};
            tail = true;
        }
        // (each thread goes over the pairs that it stored)
#pragma unroll 1
        for (int k = tid; k < (recorded ? kRayRound : 256); k += 256) {
            const u32x4 q = L.pair[k];
            const int level = (q.w & kNoBlockBit) ? -1 : (int)((q.w >> kLevelShift) & 3u);
            const bool fine = level == 0, mid = level == 1 || level == 2;
            const unsigned long long f = __ballot(fine), g = __ballot(mid);
            if (f | g) {
                uint32_t at = 0;
                if (lane == 0 && f) at = atomicAdd(&L.n[0], (uint32_t)__popcll(f));
                if (lane == 1 && g) at = atomicAdd(&L.n[1], (uint32_t)__popcll(g));
                const uint32_t a0 = (uint32_t)__builtin_amdgcn_readlane((int)at, 0), a1 = (uint32_t)__builtin_amdgcn_readlane((int)at, 1);
                if (fine) L.wait[a0 + (uint32_t)rank_in_mask(f)] = (uint16_t)k;
                if (mid) L.wait[(uint32_t)kRayRound - 1u - a1 - (uint32_t)rank_in_mask(g)] = (uint16_t)k;
            }
            if (level == 3)
                ray_coarse_block<WIDE>(m, L.seg[L.ray[k]], HashSlot{(unsigned long long)q.x | ((unsigned long long)q.y << 32), q.z, q.w}, L);
        }
        __syncthreads();
        const uint32_t n0 = uniform(L.n[0]), n1 = uniform(L.n[1]), b0 = (n0 + 63) / 64, nb = b0 + (n1 + 63) / 64;
        for (uint32_t b = (uint32_t)wv; b < nb; b += 4) {
            const bool fine = b < b0;
            const uint32_t k = (fine ? b : b - b0) * 64u + (uint32_t)lane;
            if (k < (fine ? n0 : n1)) {
                const uint32_t at = L.wait[fine ? k : (uint32_t)kRayRound - 1u - k];
                const u32x4 q = L.pair[at];
                ray_fine_block<WIDE>(m, sp.P.t, L.seg[L.ray[at]], (unsigned long long)q.x | ((unsigned long long)q.y << 32), q.z, q.w, L);
            }
        }
        __syncthreads();
    }
    touch_table_flush(m, L.touch);
    sat_table_flush(m, L.tab);
}

// Batch form of Eq. 3 and Eq. 5 for the scan's observations of one voxel: nsat at +tau, and nband
// in the band with sums s1q of q = rint(d 2^24) and Q of its squares, in square metres.  With T the former in
// metres, the band's sums of (d - D) and (d - D)^2 are T - n D and Q - 2 D T + n D^2.
__device__ inline void apply_stats(const DevMap& m, uint32_t nsat, uint32_t nband, unsigned long long s1q, double Q,
                                   float& D, uint32_t& W, float& S2) {
    const uint32_t nobs = nsat + nband;
    const double Dp = (double)D;
    const double ts = m.tau - Dp;
    const double nb = (double)nband;
    const double T = (double)(long long)s1q / kS1Scale;
    const double b2 = (Q - 2.0 * Dp * T) + nb * (Dp * Dp);
    const double s1 = (double)nsat * ts + (T - nb * Dp);
    const double s2 = (double)nsat * (ts * ts) + (b2 > 0.0 ? b2 : 0.0);
    const double Wn = (double)W + (double)nobs;
    const double S2n = (double)S2 + s2 - s1 * s1 / Wn;
    D = (float)(Dp + s1 / Wn);
    S2 = (float)(S2n > 0.0 ? S2n : 0.0);
    W = W + nobs;
}

// Read and clear one voxel's scan accumulators.
template <bool WIDE>
__device__ inline void take_accumulators(const DevMap& m, int level, size_t at, uint32_t& ns, uint32_t& nb,
                                         unsigned long long& s1, double& Q) {
    ns = m.acc_sat[level][at];
    const unsigned long long word = m.acc_s1[level][at];
    const uint32_t wide = m.band_wide ? m.acc_band[level][at] : 0u;
    band_sums(m, wide, word, nb, s1);
    Q = 0.0;
    if (ns) m.acc_sat[level][at] = 0u;
    if (nb) {
        Q = take_squares<WIDE>(m, level, at, m.acc_s2[level][at]);
        m.acc_s1[level][at] = 0ull;
        m.acc_s2[level][at] = 0ull;
        if (wide) m.acc_band[level][at] = 0u;
    }
}

// What one lane's voxels add to their block: the change of its variance sum and count, observations
// and distinct voxels.
struct UnitOut {
    double dsum = 0.0;
    int dcnt = 0, nobs = 0, distinct = 0;
};

// The scan's observations of four voxels of level-0 blocks per lane (at[k], where on[k]) into their state, the
// accumulators left at zero.  fresh: the state is empty and is written where no observation fell, too.  A
// lane owns voxels, not groups of eight, so that the lanes of a group read and write its 32 and 64 bytes
// together: with 16 bytes per lane and access the launch was bound by the L2's requests (100 M of them for
// 131072 points into an empty map: 860 us, and 702 so).  All reads of a step are issued before any is used.
constexpr int kVoxelStep = 4;
template <int ST, bool WIDE>
__device__ inline void apply_voxels(const DevMap& m, const size_t at[kVoxelStep], const bool on[kVoxelStep], bool fresh,
                                    UnitOut u[kVoxelStep]) {
    uint32_t ns[kVoxelStep], nb[kVoxelStep], W[kVoxelStep], wide[kVoxelStep];
    unsigned long long word[kVoxelStep], s1[kVoxelStep], s2[kVoxelStep];
    float D[kVoxelStep], S2[kVoxelStep];
#pragma unroll
    for (int k = 0; k < kVoxelStep; ++k) {
        ns[k] = wide[k] = W[k] = 0u, word[k] = 0ull, D[k] = S2[k] = 0.f;
        if (on[k]) {
            ns[k] = m.acc_sat[0][at[k]];
            word[k] = m.acc_s1[0][at[k]];
            if (m.band_wide) wide[k] = m.acc_band[0][at[k]];
            if (!fresh) Store<ST>::get(m, 0, at[k], D[k], W[k], S2[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < kVoxelStep; ++k) {
        band_sums(m, wide[k], word[k], nb[k], s1[k]);
        s2[k] = 0ull;
        if (nb[k]) s2[k] = m.acc_s2[0][at[k]];
    }
#pragma unroll
    for (int k = 0; k < kVoxelStep; ++k) {
        u[k] = UnitOut();
        if (ns[k] + nb[k]) {
            u[k].nobs = (int)(ns[k] + nb[k]);
            u[k].distinct = 1;
            const double before = var_term(m, W[k], S2[k]);
            const int cb = var_count(m, W[k]);
            const double Q = nb[k] ? take_squares<WIDE>(m, 0, at[k], s2[k]) : 0.0;
            apply_stats(m, ns[k], nb[k], s1[k], Q, D[k], W[k], S2[k]);
            Store<ST>::round(m, D[k], W[k], S2[k]);
            u[k].dsum = var_term(m, W[k], S2[k]) - before;
            u[k].dcnt = var_count(m, W[k]) - cb;
            if (ns[k]) m.acc_sat[0][at[k]] = 0u;
            if (nb[k]) {
                m.acc_s1[0][at[k]] = 0ull;
                m.acc_s2[0][at[k]] = 0ull;
                if (wide[k]) m.acc_band[0][at[k]] = 0u;
            }
        }
        if (fresh || u[k].distinct) Store<ST>::put(m, 0, at[k], D[k], W[k], S2[k]);
    }
}

// A block of the scan itself (level 0, one wave, lane l voxel l of each run of 64): every voxel is written,
// with zeros where no ray touched its group.
template <int ST, bool WIDE>
__device__ inline TaskOut apply_new(const DevMap& m, uint32_t id, uint32_t info, unsigned long long touched, double bvs,
                                    uint32_t bvc, int par, DeferList* dl) {
    const int lane = lane_id();
    const size_t base = (size_t)(info & kSlotMask) * 512 + (size_t)lane;
    double dsum = 0.0;
    int dcnt = 0, nobs = 0, distinct = 0;
#pragma unroll 1
    for (int r = 0; r < 8; r += kVoxelStep) {
        size_t at[kVoxelStep];
        bool on[kVoxelStep];
        UnitOut u[kVoxelStep];
        for (int k = 0; k < kVoxelStep; ++k) {
            at[k] = base + (size_t)(r + k) * 64;
            on[k] = (touched >> (8 * (r + k) + (lane >> 3))) & 1ull;
        }
        apply_voxels<ST, WIDE>(m, at, on, true, u);
        for (int k = 0; k < kVoxelStep; ++k) dsum += u[k].dsum, dcnt += u[k].dcnt, nobs += u[k].nobs, distinct += u[k].distinct;
    }
    TaskOut out;
    out.obs = out.fresh = (uint32_t)wave_sum(nobs);
    out.distinct = (uint32_t)wave_sum(distinct);
    float D[8], S2[8];  // (stored above)
    uint32_t W[8];
    (void)finish_fine<ST, true>(m, id, info, D, W, S2, true, false, (int)out.obs, dsum, dcnt, bvs, bvc, par, dl);
    return out;
}

// Blocks a task of level 0 or 1 holds at most.  A scan touches few of a block's lane groups (a ray about 5 of
// 64), so a wave takes up to kApplyBlocks blocks and gives each touched group (level 1: voxel) a lane: the chain
// of reads (queue entry, touch mask and sums, accumulators and state) is walked once for them all, where a
// wave per block walked it for every block with most of its lanes idle (131072 points on a settled map:
// 195 -> 153 us; bf16, 31 x 1023: 313 -> 241 us).
constexpr int kApplyBlocks = 8;

// Blocks per task: one until there are more blocks than kApplyWaves, then as many as keep the tasks below
// that.  With fewer tasks a launch lasts as long as one wave goes through the groups of its blocks one after
// the other: a scan of 8000 points without carving (1200 blocks of one level) 45 us with eight blocks per task, 14 with
// one.  10 waves per CU, not the 16 that it holds: the merges of a wave share their atomics (2000 points without
// carving on a street, second scan, 2900 blocks: 73 us with one block per task, 41 with two).  By the map's
// own counts, in a batch too, so that a block's sums are added in one order.
constexpr uint32_t kApplyWaves = 2560;
__device__ inline uint32_t apply_blocks_per_task(const TaskCounts& c) {
    const uint32_t n = c.n[0] + c.n[1];
    uint32_t per = 1;
    while (per < (uint32_t)kApplyBlocks && n > per * kApplyWaves) per *= 2;
    return per;
}

struct ApplyLds {  // one wave's
    unsigned long long touched[kApplyBlocks];
    double dsum[kApplyBlocks];
    uint32_t slot[kApplyBlocks];
    int dcnt[kApplyBlocks], nobs[kApplyBlocks];
    uint32_t first[kApplyBlocks + 1];
};

template <int ST, int LEVEL, bool WIDE>
__device__ inline TaskOut apply_blocks(const DevMap& m, const u32x4 MRH_GLOBAL* list, uint32_t count, uint32_t group,
                                       uint32_t per, int par, DeferList* dl, ApplyLds& A) {
    const int lane = lane_id();
    const uint32_t bi = group * per + (uint32_t)lane;
    const bool live = (uint32_t)lane < per && bi < count;
    uint32_t id = 0, info = 0, bvc = 0;
    unsigned long long touched = 0ull;
    double bvs = 0.0;
    if (live) {
        const u32x4 e = list[bi];
        id = e.x;
        info = e.y;
        touched = m.btouch[id];
        bvs = m.bvsum[id];
        bvc = m.bvcnt[id];
        m.btouch[id] = 0ull;
    }
    TaskOut out;
    const bool fresh = LEVEL == 0 && live && (info & kNewBit);
    if (LEVEL == 0) {
        for (unsigned long long left = __ballot(fresh); left; left &= left - 1ull) {
            const int j = __ffsll((long long)left) - 1;
            const TaskOut o = apply_new<ST, WIDE>(m, (uint32_t)lane_value((int)id, j), (uint32_t)lane_value((int)info, j),
                                            lane_value(touched, j), lane_value(bvs, j), (uint32_t)lane_value((int)bvc, j), par, dl);
            out.obs += o.obs;
            out.fresh += o.fresh;
            out.distinct += o.distinct;
        }
    }
    // the touched groups of the other blocks, block after block
    const bool mine = live && !fresh;
    const uint32_t n = mine ? (uint32_t)__popcll(touched) : 0u;
    uint32_t incl = n;
    for (int o = 1; o < kApplyBlocks; o <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, o);
        if (lane >= o) incl += v;
    }
    const uint32_t total = (uint32_t)lane_value((int)incl, kApplyBlocks - 1);
    if (total == 0) return out;
    if (lane < kApplyBlocks) {
        A.touched[lane] = touched;
        A.dsum[lane] = 0.0;
        A.slot[lane] = info & kSlotMask;
        A.dcnt[lane] = A.nobs[lane] = 0;
        A.first[lane + 1] = incl;
        if (lane == 0) A.first[0] = 0u;
    }
    DeferList::sync();
    int nobs = 0, distinct = 0;
    for (uint32_t base = 0; base < total; base += 64) {
        const uint32_t q = base + (uint32_t)lane;
        const bool act = q < total;
        int j = kApplyBlocks;  // (no block)
        uint32_t own = kInvalidId;  // (level 0) the lane's group, in the heap (of fewer than 2^26 slots by its size)
        UnitOut u;
        if (act) {
            j = 0;
            for (int step = kApplyBlocks / 2; step > 0; step >>= 1)
                if (q >= A.first[j + step]) j += step;
            const int g = nth_bit(A.touched[j], (int)(q - A.first[j]));
            if (LEVEL == 0) {
                own = A.slot[j] * 64u + (uint32_t)g;
            } else {
                const size_t at = (size_t)A.slot[j] * 64 + (size_t)g;
                uint32_t ns, nb, W;
                unsigned long long s1;
                double Q;
                float D, S2;
                Store<ST>::get(m, 1, at, D, W, S2);
                take_accumulators<WIDE>(m, 1, at, ns, nb, s1, Q);
                u.nobs = (int)(ns + nb);
                if (u.nobs) {
                    u.distinct = 1;
                    const double before = var_term(m, W, S2);
                    const int cb = var_count(m, W);
                    apply_stats(m, ns, nb, s1, Q, D, W, S2);
                    Store<ST>::round(m, D, W, S2);
                    u.dsum = var_term(m, W, S2) - before;
                    u.dcnt = var_count(m, W) - cb;
                    Store<ST>::put(m, 1, at, D, W, S2);
                }
            }
        }
        if (LEVEL == 0) {
            // the lanes' groups, eight at a time with a lane per voxel; a group's sums back to its lane
#pragma unroll 1
            for (int r = 0; r < 8; r += kVoxelStep) {
                if (base + 8u * (uint32_t)r >= total) break;
                size_t at[kVoxelStep];
                bool on[kVoxelStep];
                UnitOut v[kVoxelStep];
                for (int k = 0; k < kVoxelStep; ++k) {
                    const uint32_t g = (uint32_t)__shfl((int)own, 8 * (r + k) + (lane >> 3));
                    on[k] = g != kInvalidId;
                    at[k] = (size_t)g * 8 + (size_t)(lane & 7);
                }
                apply_voxels<ST, WIDE>(m, at, on, false, v);
                for (int k = 0; k < kVoxelStep; ++k) {
                    const int from = (lane & 7) * 8;
                    const double d = __shfl(group8_sum(v[k].dsum), from);
                    const int c = __shfl(group8_sum(v[k].dcnt), from), o = __shfl(group8_sum(v[k].nobs), from);
                    const int e = __shfl(group8_sum(v[k].distinct), from);
                    if ((lane >> 3) == r + k) u.dsum = d, u.dcnt = c, u.nobs = o, u.distinct = e;
                }
            }
        }
        if (act) {
            atomicAdd(&A.dcnt[j], u.dcnt);
            atomicAdd(&A.nobs[j], u.nobs);
        }
        nobs += u.nobs;
        distinct += u.distinct;
        // sums within each block's run of lanes (in lane order), added by the run's last lane
        double d = u.dsum;
        for (int o = 1; o < 64; o <<= 1) {
            const double v = __shfl_up(d, o);
            const int jo = __shfl_up(j, o);
            if (lane >= o && jo == j) d += v;
        }
        const int next = __shfl_down(j, 1);
        if (act && (lane == 63 || next != j)) A.dsum[j] += d;
        DeferList::sync();
    }
    out.obs += (uint32_t)wave_sum(nobs);
    out.distinct += (uint32_t)wave_sum(distinct);
    bool merge = false;
    if (mine) {
        const double vsum = bvs + A.dsum[lane];
        const uint32_t vcnt = bvc + (uint32_t)A.dcnt[lane];
        merge = A.nobs[lane] > 0 && LEVEL < m.levels - 1 && vcnt > 0 && vsum / (double)vcnt < m.var_thr;
        m.bvsum[id] = vsum;
        m.bvcnt[id] = vcnt;
    }
    dl->add_lanes(merge, id, info);
    DeferList::sync();
    return out;
}

// 64 / seg blocks of `level` (2: seg = 8 voxels, 3: seg = 1 voxel) per wave.
template <int ST, bool WIDE>
__device__ inline TaskOut apply_packed(const DevMap& m, const u32x4 MRH_GLOBAL* list, uint32_t count, uint32_t group, int level) {
    const int lane = lane_id();
    const int seg = level == 2 ? 8 : 1;
    const uint32_t bi = group * (uint32_t)(64 / seg) + (uint32_t)(lane / seg);
    const bool live = bi < count;
    uint32_t id = 0, info = 0, ns = 0, nb = 0;
    unsigned long long s1 = 0ull;
    double Q = 0.0;
    float D = 0.f, S2 = 0.f;
    uint32_t W = 0;
    if (live) {
        const u32x4 e = list[bi];
        id = e.x;
        info = e.y;
        const size_t at = (size_t)(info & kSlotMask) * seg + (lane % seg);
        take_accumulators<WIDE>(m, level, at, ns, nb, s1, Q);
        if (lane % seg == 0) m.btouch[id] = 0ull;
        Store<ST>::get(m, level, at, D, W, S2);
    }
    const bool upd = ns + nb > 0;
    double dsum = 0.0;
    int dcnt = 0;
    if (upd) {
        const double before = var_term(m, W, S2);
        const int cb = var_count(m, W);
        apply_stats(m, ns, nb, s1, Q, D, W, S2);
        Store<ST>::round(m, D, W, S2);
        dsum = var_term(m, W, S2) - before;
        dcnt = var_count(m, W) - cb;
    }
    TaskOut out;
    out.obs = (uint32_t)wave_sum((int)(ns + nb));
    out.distinct = (uint32_t)wave_sum(upd ? 1 : 0);
    out.merge2 = (uint32_t)wave_sum(finish_packed<ST>(m, live, id, info, level, seg, D, W, S2, upd, upd ? 1 : 0, dsum, dcnt));
    return out;
}

// A scan's update task space: [queued level-0 blocks | level-1 blocks, both in groups of apply_blocks_per_task |
// level-2 blocks in groups of 8 | level-3 blocks in groups of 64] (new blocks are queued like the others).
__device__ inline uint32_t points_task_count(const TaskCounts& c) {
    const uint32_t per = apply_blocks_per_task(c);
    return (c.n[0] + per - 1) / per + (c.n[1] + per - 1) / per + (c.n[2] + 7) / 8 + (c.n[3] + 63) / 64;
}

// One of its tasks.  Merges of level-0 / level-1 blocks are recorded in *dl, which has room for those of one
// task (DeferList::ready), and done by run_deferred.
template <int ST, bool WIDE>
__device__ inline TaskOut points_update_task(const DevMap& m, uint32_t t, const TaskCounts& c, int par, DeferList* dl,
                                             ApplyLds& A) {
    const uint32_t* n = c.n;
    const uint32_t per = apply_blocks_per_task(c), g0 = (n[0] + per - 1) / per, g1 = (n[1] + per - 1) / per;
    if (t < g0) return apply_blocks<ST, 0, WIDE>(m, m.vis[0], n[0], t, per, par, dl, A);
    t -= g0;
    if (t < g1) return apply_blocks<ST, 1, WIDE>(m, m.vis[1], n[1], t, per, par, dl, A);
    t -= g1;
    const uint32_t g2 = (n[2] + 7) / 8;
    const int level = t < g2 ? 2 : 3;
    return apply_packed<ST, WIDE>(m, m.vis[level], n[level], level == 2 ? t : t - g2, level);
}

}  // namespace mrh
