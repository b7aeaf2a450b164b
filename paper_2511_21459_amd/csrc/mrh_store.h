// Voxel-state storage formats.  Arithmetic is always FP32 in registers; these codecs convert on
// load and store (round to nearest, ties to even, for every 16-bit format).
//
//   MRH_STORE_F32   D float (m)             W uint32          S2 float (m^2)          12 B / voxel
//   MRH_STORE_F16   D half of D / tau       W uint16 (satur.) V half of S2 / (W tau^2)  6 B / voxel
//   MRH_STORE_BF16  D bfloat16 of D / tau   W half (satur.)   V half of S2 / (W tau^2)  6 B / voxel
//
// D and W of a voxel lie side by side in one plane, S2 in another: queries and meshing read D and W of
// scattered voxels, and the pair costs one read of one line (8 corners of a query point in random order
// met 2.8 lines of the pair plane on average where they met 2.3 of each of two planes).
//
// The 16-bit formats keep the per-voxel variance sigma^2 = S2 / W normalised by tau^2 rather than
// S2 itself: sigma^2 / tau^2 stays in [0, 4] whatever the weight, so it neither overflows half
// nor needs rescaling after a merge multiplies W.
#pragma once

#include <hip/hip_fp16.h>

#include <cstring>

#include "mrh_internal.h"

namespace mrh {

// float -> bfloat16, round to nearest even: the hardware conversion of gfx950 (v_cvt_pk_bf16_f32)
__device__ inline uint16_t f32_to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

__host__ __device__ inline float bf16_to_f32(uint16_t b) {
    const uint32_t u = (uint32_t)b << 16;
    float x;
    __builtin_memcpy(&x, &u, 4);
    return x;
}

__device__ inline uint16_t f32_to_f16(float x) { return __half_as_ushort(__float2half_rn(x)); }
__device__ inline float f16_to_f32(uint16_t h) { return __half2float(__ushort_as_half(h)); }

// The same conversions on the host (clang's _Float16 rounds to nearest even; bfloat16 by integer
// rounding to nearest even, NaN kept NaN).
inline float h_f16(uint16_t b) {
    _Float16 x;
    std::memcpy(&x, &b, 2);
    return (float)x;
}
inline uint16_t h_to_f16(float f) {
    const _Float16 x = (_Float16)f;
    uint16_t b;
    std::memcpy(&b, &x, 2);
    return b;
}
inline float h_bf16(uint16_t b) {
    const uint32_t u = (uint32_t)b << 16;
    float x;
    std::memcpy(&x, &u, 4);
    return x;
}
inline uint16_t h_to_bf16(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <int ST>
struct Store;

template <>
struct Store<MRH_STORE_F32> {
    __device__ static inline u32x2 MRH_GLOBAL* dw(const DevMap& m, int lvl) { return (u32x2 MRH_GLOBAL*)m.DW[lvl]; }
    __device__ static inline float MRH_GLOBAL* s2(const DevMap& m, int lvl) { return (float MRH_GLOBAL*)m.S2[lvl]; }
    // (the lanes' levels may differ)
    __device__ static inline void getDW(const DevMap& m, int lvl, size_t i, float& D, uint32_t& W) {
        const u32x2 v = ((u32x2 MRH_GLOBAL*)of_level(m.DW, lvl))[i];
        const uint32_t d = v.x;
        D = __builtin_bit_cast(float, d);
        W = v.y;
    }
    __device__ static inline void get(const DevMap& m, int lvl, size_t i, float& D, uint32_t& W, float& S2) {
        const u32x2 v = dw(m, lvl)[i];
        const uint32_t d = v.x;
        D = __builtin_bit_cast(float, d);
        W = v.y;
        S2 = s2(m, lvl)[i];
    }
    __device__ static inline void put(const DevMap& m, int lvl, size_t i, float D, uint32_t W, float S2) {
        dw(m, lvl)[i] = u32x2{__builtin_bit_cast(uint32_t, D), W};
        s2(m, lvl)[i] = S2;
    }
    __device__ static inline void round(const DevMap&, float&, uint32_t&, float&) {}
    // 8 consecutive level-0 voxels starting at base (a multiple of 8)
    __device__ static inline void get8(const DevMap& m, size_t base, float D[8], uint32_t W[8], float S2[8]) {
        u32x4 v[4];
        for (int k = 0; k < 4; ++k) v[k] = load_as<u32x4>(dw(m, 0) + base + 2 * k);
        const f32x4 s0 = load_as<f32x4>(s2(m, 0) + base), s1 = load_as<f32x4>(s2(m, 0) + base + 4);
        for (int k = 0; k < 4; ++k) {
            const uint32_t d0 = v[k].x, d1 = v[k].z;  // (a bit cast of a vector's component takes the first one)
            D[2 * k] = __builtin_bit_cast(float, d0), W[2 * k] = v[k].y;
            D[2 * k + 1] = __builtin_bit_cast(float, d1), W[2 * k + 1] = v[k].w;
        }
        S2[0] = s0.x, S2[1] = s0.y, S2[2] = s0.z, S2[3] = s0.w, S2[4] = s1.x, S2[5] = s1.y, S2[6] = s1.z, S2[7] = s1.w;
    }
    __device__ static inline void put8(const DevMap& m, size_t base, const float D[8], const uint32_t W[8],
                                       const float S2[8]) {
        for (int k = 0; k < 4; ++k)
            store_as(dw(m, 0) + base + 2 * k, u32x4{__builtin_bit_cast(uint32_t, D[2 * k]), W[2 * k],
                                                    __builtin_bit_cast(uint32_t, D[2 * k + 1]), W[2 * k + 1]});
        store_as(s2(m, 0) + base, f32x4{S2[0], S2[1], S2[2], S2[3]});
        store_as(s2(m, 0) + base + 4, f32x4{S2[4], S2[5], S2[6], S2[7]});
    }
};

// shared by the two 16-bit formats: D codec and W codec differ, the variance plane is half
template <int ST>
struct Store16 {
    __device__ static inline float decD(const DevMap& m, uint16_t b) {
        return (ST == MRH_STORE_F16 ? f16_to_f32(b) : bf16_to_f32(b)) * m.tau_f;
    }
    __device__ static inline uint16_t encD(const DevMap& m, float D) {
        const float x = D * m.inv_tau_f;
        return ST == MRH_STORE_F16 ? f32_to_f16(x) : f32_to_bf16(x);
    }
    __device__ static inline uint32_t decW(uint16_t b) {
        return ST == MRH_STORE_F16 ? (uint32_t)b : (uint32_t)f16_to_f32(b);
    }
    // u16 saturates at 65535; the half weight saturates at 65504, the largest finite half (a larger
    // W would round to infinity, whose conversion back to an integer is undefined).  A half weight
    // is exact up to 2048; above that it rounds to the nearest representable value (spacing 2 up
    // to 4096, 4 up to 8192, ...), so a single +1 observation of a voxel with W >= 2048 can leave
    // the stored weight unchanged while D and S2 still move.
    __device__ static inline uint16_t encW(uint32_t W) {
        return ST == MRH_STORE_F16 ? (uint16_t)(W < 65535u ? W : 65535u)
                                   : f32_to_f16((float)(W < 65504u ? W : 65504u));
    }
    __device__ static inline float decS2(const DevMap& m, uint16_t v, uint32_t W) {
        return f16_to_f32(v) * (float)W * m.tau2_f;
    }
    // S2 / (W tau^2) through the hardware reciprocal: the product of W and tau^2 (1/2 ulp), the
    // reciprocal (1 ulp) and the final product (1/2 ulp) keep the FP32 quotient within 2^-22 relative
    // of the exact one, against the 2^-11 relative half-ulp of the FP16 value it is rounded to
    // (an IEEE divide costs about ten instructions and this is done for every stored voxel).
    __device__ static inline uint16_t encS2(const DevMap& m, float S2, uint32_t W) {
        return f32_to_f16(W > 0 ? S2 * __builtin_amdgcn_rcpf((float)W * m.tau2_f) : 0.f);
    }
    // the values a store followed by a load gives back
    __device__ static inline void round(const DevMap& m, float& D, uint32_t& W, float& S2) {
        W = decW(encW(W));
        D = decD(m, encD(m, D));
        S2 = decS2(m, encS2(m, S2, W), W);
    }
    // a voxel's D (low half) and W in one word
    __device__ static inline uint32_t MRH_GLOBAL* dw(const DevMap& m, int lvl) { return (uint32_t MRH_GLOBAL*)m.DW[lvl]; }
    __device__ static inline uint16_t MRH_GLOBAL* s2(const DevMap& m, int lvl) { return (uint16_t MRH_GLOBAL*)m.S2[lvl]; }
    // (the lanes' levels may differ)
    __device__ static inline void getDW(const DevMap& m, int lvl, size_t i, float& D, uint32_t& W) {
        const uint32_t v = ((uint32_t MRH_GLOBAL*)of_level(m.DW, lvl))[i];
        D = decD(m, (uint16_t)v);
        W = decW((uint16_t)(v >> 16));
    }
    __device__ static inline void get(const DevMap& m, int lvl, size_t i, float& D, uint32_t& W, float& S2) {
        const uint32_t v = dw(m, lvl)[i];
        D = decD(m, (uint16_t)v);
        W = decW((uint16_t)(v >> 16));
        S2 = decS2(m, s2(m, lvl)[i], W);
    }
    __device__ static inline void put(const DevMap& m, int lvl, size_t i, float D, uint32_t W, float S2) {
        const uint16_t wb = encW(W);
        dw(m, lvl)[i] = (uint32_t)encD(m, D) | ((uint32_t)wb << 16);
        s2(m, lvl)[i] = encS2(m, S2, decW(wb));
    }
    __device__ static inline void unpack8(u32x4 v, uint16_t o[8]) {
        o[0] = (uint16_t)v.x, o[1] = (uint16_t)(v.x >> 16), o[2] = (uint16_t)v.y, o[3] = (uint16_t)(v.y >> 16);
        o[4] = (uint16_t)v.z, o[5] = (uint16_t)(v.z >> 16), o[6] = (uint16_t)v.w, o[7] = (uint16_t)(v.w >> 16);
    }
    __device__ static inline u32x4 pack8(const uint16_t o[8]) {
        return u32x4{(uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16),
                          (uint32_t)o[4] | ((uint32_t)o[5] << 16), (uint32_t)o[6] | ((uint32_t)o[7] << 16)};
    }
    __device__ static inline void get8(const DevMap& m, size_t base, float D[8], uint32_t W[8], float S2[8]) {
        const u32x4 a = load_as<u32x4>(dw(m, 0) + base), b = load_as<u32x4>(dw(m, 0) + base + 4);
        const u32x4 s = load_as<u32x4>(s2(m, 0) + base);
        const uint32_t v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint16_t sb[8];
        unpack8(s, sb);
        for (int q = 0; q < 8; ++q) {
            W[q] = decW((uint16_t)(v[q] >> 16));
            D[q] = decD(m, (uint16_t)v[q]);
            S2[q] = decS2(m, sb[q], W[q]);
        }
    }
    __device__ static inline void put8(const DevMap& m, size_t base, const float D[8], const uint32_t W[8],
                                       const float S2[8]) {
        uint32_t v[8];
        uint16_t sb[8];
        for (int q = 0; q < 8; ++q) {
            const uint16_t wb = encW(W[q]);
            v[q] = (uint32_t)encD(m, D[q]) | ((uint32_t)wb << 16);
            sb[q] = encS2(m, S2[q], decW(wb));
        }
        store_as(dw(m, 0) + base, u32x4{v[0], v[1], v[2], v[3]});
        store_as(dw(m, 0) + base + 4, u32x4{v[4], v[5], v[6], v[7]});
        store_as(s2(m, 0) + base, pack8(sb));
    }
};

template <>
struct Store<MRH_STORE_F16> : Store16<MRH_STORE_F16> {};
template <>
struct Store<MRH_STORE_BF16> : Store16<MRH_STORE_BF16> {};

// host: bytes of one element (D, W or S2)
__host__ __device__ inline int plane_bytes(int storage) { return storage == MRH_STORE_F32 ? 4 : 2; }

}  // namespace mrh
