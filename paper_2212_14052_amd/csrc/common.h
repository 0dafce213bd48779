// Device-side helpers shared by the h3flash HIP kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace h3 {

enum DType { F32 = 0, F16 = 1, BF16 = 2 };

// ------------------------------------------------------------ complex ------
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
// multiply by -i and by +i
__device__ __forceinline__ float2 cmul_mi(float2 a) { return make_float2(a.y, -a.x); }
__device__ __forceinline__ float2 cmul_pi(float2 a) { return make_float2(-a.y, a.x); }

// ------------------------------------------------------------ 16-bit I/O ---
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t b = __float_as_uint(f);
    if ((b & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((b >> 16) | 0x40u);  // quiet NaN
    b += 0x7fffu + ((b >> 16) & 1u);                                            // RNE
    return (uint16_t)(b >> 16);
}
__device__ __forceinline__ float f16_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
// float -> half conversion rounds to nearest even
__device__ __forceinline__ uint16_t f32_to_f16(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }

template <int DT> struct IO;
template <> struct IO<F32> {
    typedef float T;
    static __device__ __forceinline__ float ld(const float *p, long i) { return p[i]; }
    static __device__ __forceinline__ void st(float *p, long i, float v) { p[i] = v; }
};
template <> struct IO<F16> {
    typedef uint16_t T;
    static __device__ __forceinline__ float ld(const uint16_t *p, long i) { return f16_to_f32(p[i]); }
    static __device__ __forceinline__ void st(uint16_t *p, long i, float v) { p[i] = f32_to_f16(v); }
};
template <> struct IO<BF16> {
    typedef uint16_t T;
    static __device__ __forceinline__ float ld(const uint16_t *p, long i) { return bf16_to_f32(p[i]); }
    static __device__ __forceinline__ void st(uint16_t *p, long i, float v) { p[i] = f32_to_bf16(v); }
};

// 16-byte store of a result that nothing in this launch reads again, past the
// caches' write-allocate path: whole lines of a streaming output go out at 5.2
// TB/s beside their loads, against 4.0 with ordinary stores (a copy of 537 MB).
// For partly written lines it is slower.
__device__ __forceinline__ void store_stream(void *p, uint4 v) {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(__builtin_bit_cast(u4, v), (u4 *)p);
}

// Exponent e with m = f 2^e, f in [1/2, 1) (frexp); 0 for 0, NaN and inf, so
// that such rows pass through unscaled.
__device__ __forceinline__ int pow2_exp(float m) {
    if (!(m > 0.f) || !(m < 3.0e38f)) return 0;
    int e;
    frexpf(m, &e);
    return e;
}

// --------------------------------------------------------- launch order ----
// Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Remap
// the hardware block index so that consecutive logical indices run on the same
// XCD: work that shares data (e.g. rows of one channel) then shares an L2.
__device__ __forceinline__ int xcd_logical_block(int b, int nblocks) {
    constexpr int NXCD = 8;
    if (nblocks % NXCD != 0) return b;
    return (b % NXCD) * (nblocks / NXCD) + b / NXCD;
}

// max of x over each group of W consecutive lanes, in every lane of the group
// (W a power of two <= 64): lane exchanges on the VALU, no LDS.
template <int CTRL> __device__ __forceinline__ uint32_t max_dpp(uint32_t x) {
    const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
    return x > y ? x : y;
}
template <int W> __device__ __forceinline__ uint32_t group_max(uint32_t x) {
    if constexpr (W >= 2) x = max_dpp<0xB1>(x);     // quad_perm [1,0,3,2]
    if constexpr (W >= 4) x = max_dpp<0x4E>(x);     // quad_perm [2,3,0,1]
    if constexpr (W >= 8) x = max_dpp<0x141>(x);    // row_half_mirror
    if constexpr (W >= 16) x = max_dpp<0x140>(x);   // row_mirror
    if constexpr (W >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = r[0] > r[1] ? r[0] : r[1];
    }
    if constexpr (W >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        x = r[0] > r[1] ? r[0] : r[1];
    }
    return x;
}

// Two floats rounded to 16 bits (nearest even) in one word, lo in its low half.
template <int DT> __device__ __forceinline__ uint32_t pack_16x2(float lo, float hi) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {lo, hi};
    if constexpr (DT == BF16) {
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
    } else {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, h2));
    }
}

// Products of two 16-bit pairs, rounded once.
template <int DT> __device__ __forceinline__ uint32_t mul_16x2(uint32_t x, uint32_t z) {
    if constexpr (DT == F16) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_bit_cast(h2, x) * __builtin_bit_cast(h2, z));
    } else {
        return pack_16x2<BF16>(bf16_to_f32(x & 0xffffu) * bf16_to_f32(z & 0xffffu), bf16_to_f32(x >> 16) * bf16_to_f32(z >> 16));
    }
}

// exp(tau * lambda) for complex lambda given in float64, returned in float32:
// the phase tau*Im(lambda) is reduced modulo 2 pi in float64 before the
// float32 sine/cosine, so large arguments keep full accuracy.
__device__ __forceinline__ float2 cexp_scaled(double tau, double lre, double lim) {
    const double TWO_PI = 6.283185307179586476925286766559;
    double ph = tau * lim;
    ph -= TWO_PI * rint(ph / TWO_PI);
    float mag = expf((float)(tau * lre));
    float s, c;
    sincosf((float)ph, &s, &c);
    return make_float2(mag * c, mag * s);
}

}  // namespace h3
