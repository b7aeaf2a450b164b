// Image-space quadtree by contrast (Sec. 3.5, Eq. 10, Algorithm 1), a standalone GPU kernel set.
//
// Contrast of a node Q: the Rec. 601 luma weights l = (0.2989, 0.5870, 0.1140) times the
// per-channel mean squared deviation of its pixels' RGB values from their mean (Eq. 10).  The
// quadtree is built breadth first from the whole image: a node whose contrast exceeds the threshold
// and whose shorter side exceeds the minimum size is split at the rounded-down midpoints into
// top-left, bottom-left, top-right and bottom-right children (children without pixels dropped);
// every other node is a leaf.
//
// The paper reduces each node's pixels in shared memory, a launch per level.  Here a workgroup owns a
// node at the depth where nodes fit LDS (at most kTileSide pixels a side): it builds summed-area tables of
// its own pixels there, after which every node below costs four table reads, and it walks its subtree
// in LDS.  Which of its ancestors are split follows from their sums, which a first launch over the
// image leaves per subtree: two launches and two reads of the image whatever the depth, where tables of
// the whole image (36 B a pixel written twice and read by every level) took three and one per level.
// Long thin images and the longest ones keep those tables (mrh_quadtree_build has the rule).
// With S_c and Q_c a node's sums of channel values and of their squares over its n pixels (exact
// integers), n^2 times the channel variance is n Q_c - S_c^2, exact in 64 bits for images of up to
// 2^23 pixels; the contrast is then formed in FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>

#include "mrhash.h"

namespace {

constexpr int64_t kMaxPixels = int64_t(1) << 23;
constexpr int kMaxLevels = 32;  // levels of the breadth-first build (at most log2(2^23) + 3 are used)

struct QtNode {
    int32_t x, y, w, h;
};

// Row pass: inclusive prefix sums along x of each channel and of its square, written at (y + 1,
// x + 1) of (H + 1) x (W + 1) planes whose row 0 and column 0 are zero.  One workgroup per row.
// Workgroup 0 also sets up the breadth-first build: the root node in the first queue, one node at
// level 0, none at the other levels and no leaves (counts: kMaxLevels level counts, then the u64
// leaf count).
__global__ __launch_bounds__(256) void k_sat_rows(const uint8_t* __restrict__ rgb, int32_t W, int32_t H,
                                                  uint32_t* __restrict__ S, unsigned long long* __restrict__ Q,
                                                  QtNode* __restrict__ queue0, uint32_t* __restrict__ counts) {
    const int32_t y = blockIdx.x;
    if (y == 0) {
        if (threadIdx.x == 0) queue0[0] = QtNode{0, 0, W, H};
        if (threadIdx.x < kMaxLevels + 2) counts[threadIdx.x] = threadIdx.x == 0 ? 1u : 0u;
    }
    const size_t pitch = (size_t)W + 1, plane = pitch * ((size_t)H + 1);
    const int per = (W + 255) / 256;
    const int x0 = threadIdx.x * per, x1 = min(W, x0 + per);
    uint32_t s[3] = {0, 0, 0};
    unsigned long long q[3] = {0, 0, 0};
    for (int x = x0; x < x1; ++x)
        for (int c = 0; c < 3; ++c) {
            const uint32_t v = rgb[3 * ((size_t)y * W + x) + c];
            s[c] += v;
            q[c] += (unsigned long long)(v * v);
        }
    __shared__ uint32_t ss[3][256];
    __shared__ unsigned long long sq[3][256];
    for (int c = 0; c < 3; ++c) ss[c][threadIdx.x] = s[c], sq[c][threadIdx.x] = q[c];
    __syncthreads();
    // inclusive scan of the per-thread totals (Hillis-Steele, 256 entries)
    for (int o = 1; o < 256; o <<= 1) {
        uint32_t a[3] = {0, 0, 0};
        unsigned long long b[3] = {0, 0, 0};
        if ((int)threadIdx.x >= o)
            for (int c = 0; c < 3; ++c) a[c] = ss[c][threadIdx.x - o], b[c] = sq[c][threadIdx.x - o];
        __syncthreads();
        for (int c = 0; c < 3; ++c) ss[c][threadIdx.x] += a[c], sq[c][threadIdx.x] += b[c];
        __syncthreads();
    }
    for (int c = 0; c < 3; ++c) {
        s[c] = threadIdx.x ? ss[c][threadIdx.x - 1] : 0u;
        q[c] = threadIdx.x ? sq[c][threadIdx.x - 1] : 0ull;
    }
    const size_t row = ((size_t)y + 1) * pitch;
    for (int x = x0; x < x1; ++x)
        for (int c = 0; c < 3; ++c) {
            const uint32_t v = rgb[3 * ((size_t)y * W + x) + c];
            s[c] += v;
            q[c] += (unsigned long long)(v * v);
            S[c * plane + row + x + 1] = s[c];
            Q[c * plane + row + x + 1] = q[c];
        }
    if (threadIdx.x < 3) {
        S[threadIdx.x * plane + row] = 0u;
        Q[threadIdx.x * plane + row] = 0ull;
    }
}

// Column pass: running sums down each column, in chunks of kColChunk rows so that the image's
// height is covered by many threads (consecutive threads take consecutive columns, so every row
// access is coalesced): the chunks' column sums, then the running sums within each chunk, started
// from the sum of the chunks above it (read together, independent loads).
constexpr int kColChunk = 16;

__global__ __launch_bounds__(64) void k_sat_cols_part(int32_t W, int32_t H, const uint32_t* __restrict__ S,
                                                      const unsigned long long* __restrict__ Q, uint32_t* __restrict__ TS,
                                                      unsigned long long* __restrict__ TQ) {
    const int32_t x = blockIdx.x * blockDim.x + threadIdx.x, k = blockIdx.y;
    if (x > W) return;
    const size_t pitch = (size_t)W + 1, plane = pitch * ((size_t)H + 1);
    const int32_t y0 = k * kColChunk + 1, y1 = min(H, y0 + kColChunk - 1);
    for (int c = 0; c < 3; ++c) {
        uint32_t s = 0;
        unsigned long long q = 0;
#pragma unroll
        for (int32_t r = 0; r < kColChunk; ++r) {
            const int32_t y = y0 + r;
            const size_t at = c * plane + (size_t)y * pitch + x;
            s += y <= y1 ? S[at] : 0u;
            q += y <= y1 ? Q[at] : 0ull;
        }
        TS[((size_t)k * 3 + c) * pitch + x] = s;
        TQ[((size_t)k * 3 + c) * pitch + x] = q;
    }
}

__global__ __launch_bounds__(64) void k_sat_cols_apply(int32_t W, int32_t H, uint32_t* __restrict__ S,
                                                       unsigned long long* __restrict__ Q, const uint32_t* __restrict__ TS,
                                                       const unsigned long long* __restrict__ TQ) {
    const int32_t x = blockIdx.x * blockDim.x + threadIdx.x, k = blockIdx.y;
    if (x > W) return;
    const size_t pitch = (size_t)W + 1, plane = pitch * ((size_t)H + 1);
    const int32_t y0 = k * kColChunk + 1, y1 = min(H, y0 + kColChunk - 1);
    for (int c = 0; c < 3; ++c) {
        if (k == 0) {
            S[c * plane + x] = 0u;
            Q[c * plane + x] = 0ull;
        }
        uint32_t s = 0;
        unsigned long long q = 0;
#pragma unroll 8
        for (int32_t j = 0; j < k; ++j) {
            s += TS[((size_t)j * 3 + c) * pitch + x];
            q += TQ[((size_t)j * 3 + c) * pitch + x];
        }
        // the chunk's rows read first (independent loads), then the running sums written
        uint32_t rs[kColChunk];
        unsigned long long rq[kColChunk];
#pragma unroll
        for (int32_t r = 0; r < kColChunk; ++r) {
            const int32_t y = y0 + r;
            const size_t at = c * plane + (size_t)y * pitch + x;
            rs[r] = y <= y1 ? S[at] : 0u;
            rq[r] = y <= y1 ? Q[at] : 0ull;
        }
#pragma unroll
        for (int32_t r = 0; r < kColChunk; ++r) {
            const int32_t y = y0 + r;
            if (y > y1) break;
            const size_t at = c * plane + (size_t)y * pitch + x;
            s += rs[r];
            q += rq[r];
            S[at] = s;
            Q[at] = q;
        }
    }
}

// Eq. 10 from the exact sums of a node's n pixels.
__device__ inline double contrast_of(unsigned long long n, const unsigned long long sum[3], const unsigned long long sq[3]) {
    const double l[3] = {0.2989, 0.5870, 0.1140};
    double con = 0.0;
    for (int k = 0; k < 3; ++k) {
        const unsigned long long v = n * sq[k] - sum[k] * sum[k];  // n^2 times the channel variance, exact
        con += l[k] * (double)v;
    }
    return con / ((double)n * (double)n);
}

__device__ inline double node_contrast(const uint32_t* S, const unsigned long long* Q, int32_t W, int32_t H,
                                       const QtNode& nd) {
    const size_t pitch = (size_t)W + 1, plane = pitch * ((size_t)H + 1);
    const size_t a = (size_t)nd.y * pitch + nd.x, b = a + nd.w, c = ((size_t)nd.y + nd.h) * pitch + nd.x, d = c + nd.w;
    unsigned long long sum[3], sq[3];
    for (int k = 0; k < 3; ++k) {
        const uint32_t* s = S + k * plane;
        const unsigned long long* q = Q + k * plane;
        sum[k] = (unsigned long long)(s[d] - s[b] - s[c] + s[a]);
        sq[k] = q[d] - q[b] - q[c] + q[a];
    }
    return contrast_of((unsigned long long)nd.w * (unsigned long long)nd.h, sum, sq);
}

// One breadth-first level: every node of the input queue is split into the output queue or written
// as a leaf (wave-aggregated appends).
__global__ __launch_bounds__(256) void k_qt_level(const uint32_t* __restrict__ S, const unsigned long long* __restrict__ Q,
                                                  int32_t W, int32_t H, double threshold, int32_t min_size,
                                                  const QtNode* __restrict__ in, const uint32_t* __restrict__ n_in,
                                                  QtNode* __restrict__ out, uint32_t* __restrict__ n_out,
                                                  int32_t* leaves, float* contrast, unsigned long long* n_leaves,
                                                  long long cap) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t count = *n_in;
    QtNode kids[4];
    int nk = 0;
    bool leaf = false;
    double con = 0.0;
    QtNode nd{0, 0, 0, 0};
    if (i < count) {
        nd = in[i];
        con = node_contrast(S, Q, W, H, nd);
        if (con > threshold && min(nd.w, nd.h) > min_size) {
            const int32_t wl = nd.w / 2, ht = nd.h / 2;
            const QtNode cand[4] = {{nd.x, nd.y, wl, ht}, {nd.x, nd.y + ht, wl, nd.h - ht},
                                    {nd.x + wl, nd.y, nd.w - wl, ht}, {nd.x + wl, nd.y + ht, nd.w - wl, nd.h - ht}};
            for (int k = 0; k < 4; ++k)
                if (cand[k].w > 0 && cand[k].h > 0) kids[nk++] = cand[k];
        } else {
            leaf = true;
        }
    }
    // children: per-lane counts, one atomic per wave
    const int lane = __lane_id();
    int incl = nk;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    const int wtot = __shfl(incl, 63);
    uint32_t base = 0;
    if (lane == 63 && wtot) base = atomicAdd(n_out, (uint32_t)wtot);
    base = (uint32_t)__shfl((int)base, 63);
    for (int k = 0; k < nk; ++k) out[base + (uint32_t)(incl - nk + k)] = kids[k];
    const unsigned long long lm = __ballot(leaf);
    if (lm) {
        unsigned long long lb = 0;
        const int first = __ffsll((long long)lm) - 1;
        if (lane == first) lb = atomicAdd(n_leaves, (unsigned long long)__popcll(lm));
        lb = ((unsigned long long)__shfl((int)(uint32_t)(lb >> 32), first) << 32) | (uint32_t)__shfl((int)(uint32_t)lb, first);
        if (leaf) {
            const long long at = (long long)(lb + (unsigned long long)__builtin_amdgcn_mbcnt_hi(
                                                        (uint32_t)(lm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lm, 0)));
            if (at < cap) {
                if (leaves) {
                    leaves[4 * at] = nd.x;
                    leaves[4 * at + 1] = nd.y;
                    leaves[4 * at + 2] = nd.w;
                    leaves[4 * at + 3] = nd.h;
                }
                if (contrast) contrast[at] = (float)con;
            }
        }
    }
}

// ---- subtrees in LDS --------------------------------------------------------------------------

constexpr int kTileSide = 40;    // longest side of a subtree's root (640 x 480: 256 workgroups of 40 x 30)
constexpr int kTilePitch = kTileSide + 1;
constexpr int kTilePixels = kTileSide * kTileSide;
constexpr int kTileDepth = 7;    // deepest subtree root
constexpr int64_t kDeepPixels = 2500000;  // images from which subtree roots may lie that deep
constexpr int kTileThreads = 512;

// Sums of a node's channel values and squares.
struct QtSums {
    unsigned long long q[3];
    uint32_t s[3], unused;
};

// Node `path` (two bits per level, the split's order: bit 1 right, bit 0 bottom) of depth d.
__device__ inline QtNode node_at(int32_t W, int32_t H, int d, uint32_t path) {
    QtNode nd{0, 0, W, H};
    for (int k = d - 1; k >= 0; --k) {
        const uint32_t b = path >> (2 * k);
        const int32_t wl = nd.w / 2, ht = nd.h / 2;
        if (b & 2u) nd.x += wl, nd.w -= wl;
        else nd.w = wl;
        if (b & 1u) nd.y += ht, nd.h -= ht;
        else nd.h = ht;
    }
    return nd;
}

__host__ __device__ inline size_t sums_at(int d) { return ((size_t(1) << (2 * d)) - 1) / 3; }  // nodes above depth d

__device__ inline void add_xor(QtSums& v, int lane) {
    for (int c = 0; c < 3; ++c) {
        v.s[c] += (uint32_t)__shfl_xor((int)v.s[c], lane);
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v.q[c], lane);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v.q[c] >> 32), lane);
        v.q[c] += ((unsigned long long)hi << 32) | lo;
    }
}

// Sums of the subtree roots, one workgroup each: a read of the image, 4 us at 640 x 480.  Workgroup 0
// clears the leaf count.
__global__ __launch_bounds__(256) void k_qt_sums(const uint8_t* __restrict__ rgb, int32_t W, int32_t H, int depth,
                                                 QtSums* __restrict__ sums, unsigned long long* __restrict__ n_leaves) {
    const uint32_t path = blockIdx.x;
    if (path == 0 && threadIdx.x == 0) *n_leaves = 0ull;
    const QtNode nd = node_at(W, H, depth, path);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t s[3] = {0, 0, 0}, q[3] = {0, 0, 0};  // (a subtree's squares fit 32 bits: kTilePixels x 255^2)
    static_assert((uint64_t)kTilePixels * 255 * 255 < (uint64_t(1) << 32), "subtree sums in 32 bits");
    if (lane < nd.w) {
        const uint8_t* p = rgb + 3 * ((size_t)nd.y * W + nd.x + lane);
        uint32_t v[3][kTileSide / 4];  // every row's reads in flight together
#pragma unroll
        for (int i = 0; i < kTileSide / 4; ++i)
            for (int c = 0; c < 3; ++c) v[c][i] = wave + 4 * i < nd.h ? p[3 * (size_t)(wave + 4 * i) * W + c] : 0u;
#pragma unroll
        for (int i = 0; i < kTileSide / 4; ++i)
            for (int c = 0; c < 3; ++c) s[c] += v[c][i], q[c] += v[c][i] * v[c][i];
    }
    for (int o = 1; o < 64; o <<= 1)
        for (int c = 0; c < 3; ++c) {
            s[c] += (uint32_t)__shfl_xor((int)s[c], o);
            q[c] += (uint32_t)__shfl_xor((int)q[c], o);
        }
    __shared__ uint32_t part[4][6];
    if (lane == 0)
        for (int c = 0; c < 3; ++c) part[wave][c] = s[c], part[wave][3 + c] = q[c];
    __syncthreads();
    if (threadIdx.x) return;
    QtSums o{};
    for (int w = 0; w < 4; ++w)
        for (int c = 0; c < 3; ++c) o.s[c] += part[w][c], o.q[c] += part[w][3 + c];
    sums[sums_at(depth) + path] = o;
}

// Sums of the nodes at depths depth - 4 .. depth - 1 (subtree roots deeper than 4 only): a workgroup per
// node of depth - 4, a thread per subtree root below it.
__global__ __launch_bounds__(256) void k_qt_reduce(int depth, QtSums* __restrict__ sums) {
    const uint32_t t = threadIdx.x, path = blockIdx.x * 256 + t;
    QtSums v = sums[sums_at(depth) + path];
    for (int j = 1; j <= 3; ++j) {
        add_xor(v, 1 << (2 * j - 2));
        add_xor(v, 2 << (2 * j - 2));
        if ((t & ((1u << (2 * j)) - 1u)) == 0) sums[sums_at(depth - j) + (path >> (2 * j))] = v;
    }
    __shared__ QtSums part[4];
    if ((t & 63u) == 0) part[t >> 6] = v;
    __syncthreads();
    if (t) return;
    for (int w = 1; w < 4; ++w)
        for (int c = 0; c < 3; ++c) v.s[c] += part[w].s[c], v.q[c] += part[w].q[c];
    sums[sums_at(depth - 4) + blockIdx.x] = v;
}

struct QtLds {
    uint32_t table[6][kTilePitch * kTilePitch];  // sums of the subtree's channels, then of their squares
    uint32_t queue[2][kTilePixels];              // nodes of a level (x, y, w, h in six bits each)
    uint32_t leaf[kTilePixels];
    float contrast[kTilePixels];
    QtSums above[kTileDepth];                    // the subtree root's ancestors
    QtSums part[4];
    int first_leaf;                              // depth of the first ancestor that is a leaf (depth: none)
    uint32_t n[3], n_leaf;                       // queue lengths by level modulo 3
    unsigned long long base;
};

// Leaves of the subtree below node blockIdx.x of `depth`.  The levels are a chain of table reads and
// barriers in LDS, and one append to the leaf list per workgroup (its order is free).  An ancestor
// that is a leaf is written by the last of the workgroups below it.  640 x 480, 34957 leaves, a build with
// its read-back: 176 -> 43 us, of which half is the host's.
__global__ __launch_bounds__(kTileThreads) void k_qt_tree(const uint8_t* __restrict__ rgb, int32_t W, int32_t H, int depth,
                                                          const QtSums* __restrict__ sums, double threshold,
                                                          int32_t min_size, int32_t* leaves, float* contrast,
                                                          unsigned long long* n_leaves, long long cap) {
    __shared__ QtLds L;
    const uint32_t path = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    constexpr int kWaves = kTileThreads / 64, kRows = kTileSide / kWaves;
    static_assert(kTileSide % kWaves == 0 && kTileSide < 64, "a wave takes whole rows");
    const QtNode nd = node_at(W, H, depth, path);

    // the subtree's pixels (used after the ancestors' sums: in flight meanwhile)
    uint32_t v[kRows][3];
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int y = wave + i * kWaves;
        const bool in = lane < nd.w && y < nd.h;
        const uint8_t* p = rgb + (in ? 3 * ((size_t)(nd.y + y) * W + nd.x + lane) : 0);
        for (int c = 0; c < 3; ++c) v[i][c] = in ? p[c] : 0u;
    }

    // ancestors: those below depth `top` read, the others summed from the nodes of depth `top`
    const int top = depth > 4 ? depth - 4 : depth;
    if (t < 256) {
        QtSums a{};
        if (t < 1 << (2 * top)) a = sums[sums_at(top) + t];
        for (int j = 1; j <= 3; ++j) {
            add_xor(a, 1 << (2 * j - 2));
            add_xor(a, 2 << (2 * j - 2));
            const int d = top - j;
            if (d >= 0 && (uint32_t)t == (path >> (2 * (depth - d))) << (2 * j)) L.above[d] = a;
        }
        if (lane == 0) L.part[wave] = a;
    } else if (t - 256 < depth - top) {
        const int d = top + t - 256;
        L.above[d] = sums[sums_at(d) + (path >> (2 * (depth - d)))];
    }
    if (t < 3) L.n[t] = t == 0 ? 1u : 0u;
    if (t == 3) L.n_leaf = 0u;
    if (t == 4) L.queue[0][0] = (uint32_t)nd.w << 12 | (uint32_t)nd.h << 18;
    __syncthreads();
    if (wave == 0) {
        bool leaf = false;
        double con = 0.0;
        QtNode an{};
        if (lane < depth) {
            QtSums a = L.above[lane];
            if (top == 4 && lane == 0) {
                a = L.part[0];
                for (int w = 1; w < 4; ++w)
                    for (int c = 0; c < 3; ++c) a.s[c] += L.part[w].s[c], a.q[c] += L.part[w].q[c];
            }
            an = node_at(W, H, lane, path >> (2 * (depth - lane)));
            const unsigned long long sum[3] = {a.s[0], a.s[1], a.s[2]};
            if (an.w > 0 && an.h > 0) con = contrast_of((unsigned long long)an.w * (unsigned long long)an.h, sum, a.q);
            leaf = !(con > threshold && min(an.w, an.h) > min_size);
        }
        const unsigned long long m = __ballot(leaf);
        const int f = m ? __ffsll((long long)m) - 1 : depth;
        if (lane == 0) L.first_leaf = f;
        const uint32_t below = (1u << (2 * (depth - f))) - 1u;
        if (lane == f && f < depth && (path & below) == below) {
            const long long at = (long long)atomicAdd(n_leaves, 1ull);
            if (at < cap) {
                if (leaves) {
                    leaves[4 * at] = an.x;
                    leaves[4 * at + 1] = an.y;
                    leaves[4 * at + 2] = an.w;
                    leaves[4 * at + 3] = an.h;
                }
                if (contrast) contrast[at] = (float)con;
            }
        }
    }
    __syncthreads();
    if (L.first_leaf < depth) return;

    // summed-area tables: rows by shuffles, then columns
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int y = wave + i * kWaves;
        uint32_t s0 = v[i][0], s1 = v[i][1], s2 = v[i][2];
        uint32_t q0 = v[i][0] * v[i][0], q1 = v[i][1] * v[i][1], q2 = v[i][2] * v[i][2];
        for (int o = 1; o < kTileSide; o <<= 1) {
            const uint32_t a = (uint32_t)__shfl_up((int)s0, o), b = (uint32_t)__shfl_up((int)s1, o);
            const uint32_t d = (uint32_t)__shfl_up((int)s2, o);
            const uint32_t e = (uint32_t)__shfl_up((int)q0, o), f = (uint32_t)__shfl_up((int)q1, o);
            const uint32_t g = (uint32_t)__shfl_up((int)q2, o);
            if (lane >= o) s0 += a, s1 += b, s2 += d, q0 += e, q1 += f, q2 += g;
        }
        if (lane < nd.w && y < nd.h) {
            const int at = (y + 1) * kTilePitch + lane + 1;
            L.table[0][at] = s0;
            L.table[1][at] = s1;
            L.table[2][at] = s2;
            L.table[3][at] = q0;
            L.table[4][at] = q1;
            L.table[5][at] = q2;
        }
    }
    __syncthreads();
    if (t < 6 * kTilePitch) {
        const int plane = t / kTilePitch, x = t % kTilePitch;
        if (x <= nd.w) {
            uint32_t* col = L.table[plane] + x;
            uint32_t sum = 0;
            col[0] = 0u;
            for (int y = 1; y <= nd.h; ++y) {
                sum += x ? col[y * kTilePitch] : 0u;
                col[y * kTilePitch] = sum;
            }
        }
    }
    static_assert(6 * kTilePitch <= kTileThreads, "a thread per column and plane");
    __syncthreads();

    // (split sides are above min_size >= 1, so every child has pixels)
    for (int d = 0;; ++d) {
        const uint32_t count = L.n[d % 3];
        if (!count) break;
        const uint32_t* in = L.queue[d & 1];
        uint32_t* out = L.queue[(d & 1) ^ 1];
        if (t == 0) L.n[(d + 2) % 3] = 0u;
        for (uint32_t i0 = (uint32_t)wave * 64u; i0 < count; i0 += kTileThreads) {
            const uint32_t i = i0 + lane;
            bool leaf = false, split = false;
            uint32_t x = 0, y = 0, w = 0, h = 0;
            double con = 0.0;
            if (i < count) {
                const uint32_t k = in[i];
                x = k & 63u, y = k >> 6 & 63u, w = k >> 12 & 63u, h = k >> 18;
                const uint32_t a = y * kTilePitch + x, c = (y + h) * kTilePitch + x;
                unsigned long long sum[6];
                for (int p = 0; p < 6; ++p) {
                    const uint32_t* s = L.table[p];
                    sum[p] = s[c + w] - s[a + w] - s[c] + s[a];
                }
                con = contrast_of((unsigned long long)(w * h), sum, sum + 3);
                split = con > threshold && (int32_t)min(w, h) > min_size;
                leaf = !split;
            }
            const unsigned long long below = (1ull << lane) - 1ull, ml = __ballot(leaf), ms = __ballot(split);
            uint32_t bl = 0, bs = 0;
            if (lane == 0) {
                if (ml) bl = atomicAdd(&L.n_leaf, (uint32_t)__popcll(ml));
                if (ms) bs = atomicAdd(&L.n[(d + 1) % 3], 4u * (uint32_t)__popcll(ms));
            }
            bl = (uint32_t)__builtin_amdgcn_readfirstlane((int)bl);
            bs = (uint32_t)__builtin_amdgcn_readfirstlane((int)bs);
            if (leaf) {
                const uint32_t at = bl + (uint32_t)__popcll(ml & below);
                L.leaf[at] = x | y << 6 | w << 12 | h << 18;
                L.contrast[at] = (float)con;
            }
            if (split) {
                const uint32_t at = bs + 4u * (uint32_t)__popcll(ms & below), wl = w / 2, ht = h / 2;
                out[at] = x | y << 6 | wl << 12 | ht << 18;
                out[at + 1] = x | (y + ht) << 6 | wl << 12 | (h - ht) << 18;
                out[at + 2] = (x + wl) | y << 6 | (w - wl) << 12 | ht << 18;
                out[at + 3] = (x + wl) | (y + ht) << 6 | (w - wl) << 12 | (h - ht) << 18;
            }
        }
        __syncthreads();
    }
    const uint32_t n = L.n_leaf;
    if (t == 0) L.base = atomicAdd(n_leaves, (unsigned long long)n);
    __syncthreads();
    for (uint32_t i = t; i < n; i += kTileThreads) {
        const long long at = (long long)(L.base + i);
        if (at >= cap) break;
        const uint32_t k = L.leaf[i];
        if (leaves) {
            leaves[4 * at] = nd.x + (int32_t)(k & 63u);
            leaves[4 * at + 1] = nd.y + (int32_t)(k >> 6 & 63u);
            leaves[4 * at + 2] = (int32_t)(k >> 12 & 63u);
            leaves[4 * at + 3] = (int32_t)(k >> 18);
        }
        if (contrast) contrast[at] = L.contrast[i];
    }
}

// Depth of the subtree roots: the shallowest whose sides are at most kTileSide (halves round up).
int tile_depth(int32_t longer) {
    int d = 0;
    for (; longer > kTileSide; longer = (longer + 1) / 2) ++d;
    return d;
}

}  // namespace

struct mrh_quadtree {
    hipStream_t stream = nullptr;
    int32_t max_w = 0, max_h = 0;
    uint32_t* S = nullptr;
    unsigned long long* Q = nullptr;
    QtNode* queue[2] = {nullptr, nullptr};
    uint32_t* counts = nullptr;  // queue length of every level (kMaxLevels), then the leaf count (u64)
    unsigned long long* n_leaves = nullptr;
    size_t queue_cap = 0;
    uint32_t* TS = nullptr;      // column pass: per chunk of rows, channel and column
    unsigned long long* TQ = nullptr;
    QtSums* sums = nullptr;      // nodes of depths 0 .. the subtree roots'
};

extern "C" {

mrh_status mrh_quadtree_create(int32_t max_width, int32_t max_height, void* stream, mrh_quadtree** out) {
    if (!out || max_width < 1 || max_height < 1 || (int64_t)max_width * max_height > kMaxPixels) return MRH_ERR_INVALID_ARG;
    *out = nullptr;
    mrh_quadtree* q = new mrh_quadtree();
    q->stream = static_cast<hipStream_t>(stream);
    q->max_w = max_width;
    q->max_h = max_height;
    const size_t plane = ((size_t)max_width + 1) * ((size_t)max_height + 1);
    // a level never holds more nodes than pixels
    q->queue_cap = (size_t)max_width * (size_t)max_height;
    const size_t chunks = ((size_t)max_height + kColChunk - 1) / kColChunk;
    bool ok = hipMalloc((void**)&q->S, 3 * plane * 4) == hipSuccess && hipMalloc((void**)&q->Q, 3 * plane * 8) == hipSuccess &&
              hipMalloc((void**)&q->queue[0], q->queue_cap * sizeof(QtNode)) == hipSuccess &&
              hipMalloc((void**)&q->queue[1], q->queue_cap * sizeof(QtNode)) == hipSuccess &&
              hipMalloc((void**)&q->counts, kMaxLevels * 4 + 8) == hipSuccess &&
              hipMalloc((void**)&q->TS, chunks * 3 * ((size_t)max_width + 1) * 4) == hipSuccess &&
              hipMalloc((void**)&q->TQ, chunks * 3 * ((size_t)max_width + 1) * 8) == hipSuccess &&
              hipMalloc((void**)&q->sums, sums_at(std::min(kTileDepth, tile_depth(std::max(max_width, max_height))) + 1) *
                                              sizeof(QtSums)) == hipSuccess;
    if (ok) q->n_leaves = reinterpret_cast<unsigned long long*>(q->counts + kMaxLevels);
    if (!ok) {
        (void)hipGetLastError();
        mrh_quadtree_destroy(q);
        return MRH_ERR_OOM;
    }
    *out = q;
    return MRH_OK;
}

void mrh_quadtree_destroy(mrh_quadtree* q) {
    if (!q) return;
    if (q->stream) (void)hipStreamSynchronize(q->stream);
    else (void)hipDeviceSynchronize();
    void* ptrs[] = {q->S, q->Q, q->queue[0], q->queue[1], q->counts, q->TS, q->TQ, q->sums};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    delete q;
}

mrh_status mrh_quadtree_build(mrh_quadtree* q, const uint8_t* rgb_dev, int32_t width, int32_t height, double threshold,
                              int32_t min_size, int32_t* leaves_dev, float* contrast_dev, int64_t cap, int64_t* n_leaves) {
    if (!q || !rgb_dev || !n_leaves || width < 1 || height < 1 || width > q->max_w || height > q->max_h || min_size < 1 ||
        cap < 0 || !(threshold == threshold))
        return MRH_ERR_INVALID_ARG;
    hipStream_t s = q->stream;
    const long long room = leaves_dev || contrast_dev ? cap : 0;
    const int32_t longer = std::max(width, height), shorter = std::min(width, height);
    const int tiles = tile_depth(longer);
    // Subtrees in LDS, unless the longer side asks for more subtree roots than the chip holds at once
    // (256 at depth 4) and the shorter one leaves most of them nearly empty, or there are so many
    // (16384 at depth 7, four times as many one deeper) that they take longer than the tables, whose time goes
    // with the pixels.  Whole builds, against the tables of the whole image: 640 x 480 69 us to 217,
    // 641 x 480 (depth 5) 89 to 215, 1281 x 240 (6) 151 to 192, 2560 x 1440 186 to 571; depth 7: 2561 x 800 422 to
    // 391, 3800 x 480 415 to 372, but 2561 x 1000 426 to 438, 3800 x 640 421 to 444, 5120 x 640 423 to 559;
    // depth 8: 5121 x 800 1514 to 644, 5121 x 1600 1547 to 1242.
    const bool deep_enough = tiles < kTileDepth || (tiles == kTileDepth && (int64_t)width * height >= kDeepPixels);
    if (tiles <= 4 || (deep_enough && longer <= 8ll * shorter)) {
        hipLaunchKernelGGL(k_qt_sums, dim3(1u << (2 * tiles)), dim3(256), 0, s, rgb_dev, width, height, tiles, q->sums,
                           q->n_leaves);
        if (tiles > 4) hipLaunchKernelGGL(k_qt_reduce, dim3(1u << (2 * (tiles - 4))), dim3(256), 0, s, tiles, q->sums);
        hipLaunchKernelGGL(k_qt_tree, dim3(1u << (2 * tiles)), dim3(kTileThreads), 0, s, rgb_dev, width, height, tiles,
                           q->sums, threshold, min_size, leaves_dev, contrast_dev, q->n_leaves, room);
    } else {
        // the summed-area tables; the row pass also puts the root in the first queue and clears the counts
        hipLaunchKernelGGL(k_sat_rows, dim3(height), dim3(256), 0, s, rgb_dev, width, height, q->S, q->Q, q->queue[0],
                           q->counts);
        const int32_t chunks = (height + kColChunk - 1) / kColChunk;
        const dim3 cg((unsigned)((width + 1 + 63) / 64), (unsigned)chunks);
        hipLaunchKernelGGL(k_sat_cols_part, cg, dim3(64), 0, s, width, height, q->S, q->Q, q->TS, q->TQ);
        hipLaunchKernelGGL(k_sat_cols_apply, cg, dim3(64), 0, s, width, height, q->S, q->Q, q->TS, q->TQ);
        // levels: a node's shorter side halves at each split, so the tree is at most
        // log2(min(width, height)) + 2 levels deep
        int depth = 1;
        for (int32_t side = std::min(width, height); side > 1; side = (side + 1) / 2) ++depth;
        const int64_t pixels = (int64_t)width * height;
        int64_t bound = 1;
        for (int d = 0; d <= depth; ++d) {
            const int cur = d & 1;
            const unsigned grid = (unsigned)((std::min(bound, pixels) + 255) / 256);
            hipLaunchKernelGGL(k_qt_level, dim3(grid), dim3(256), 0, s, q->S, q->Q, width, height, threshold, min_size,
                               q->queue[cur], q->counts + d, q->queue[cur ^ 1], q->counts + d + 1, leaves_dev,
                               contrast_dev, q->n_leaves, room);
            bound *= 4;
        }
    }
    if (hipGetLastError() != hipSuccess) return MRH_ERR_HIP;
    unsigned long long n = 0;
    if (hipMemcpyAsync(&n, q->n_leaves, 8, hipMemcpyDeviceToHost, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return MRH_ERR_HIP;
    *n_leaves = (int64_t)n;
    if ((leaves_dev || contrast_dev) && (int64_t)n > cap) return MRH_ERR_BUFFER_TOO_SMALL;
    return MRH_OK;
}

}  // extern "C"
