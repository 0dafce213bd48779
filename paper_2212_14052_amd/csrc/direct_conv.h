// Shared by the kernels that convolve 16-bit rows by direct summation on the
// matrix cores: 16x16x32 products, 16-bit pairs, and operands whose elements
// start at any 16-bit offset of an LDS array.
#pragma once
#include "common.h"

namespace h3 {

typedef _Float16 cd_h8 __attribute__((ext_vector_type(8)));
typedef __bf16 cd_b8 __attribute__((ext_vector_type(8)));
typedef _Float16 cd_h2 __attribute__((ext_vector_type(2)));
typedef __bf16 cd_b2 __attribute__((ext_vector_type(2)));
typedef unsigned cd_u4 __attribute__((ext_vector_type(4)));
typedef float cd_f2 __attribute__((ext_vector_type(2)));
typedef float cd_f4 __attribute__((ext_vector_type(4)));

template <int DT>
__device__ __forceinline__ cd_f4 cd_mfma(uint4 a, uint4 b, cd_f4 c) {
    if constexpr (DT == BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(cd_b8, a), __builtin_bit_cast(cd_b8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(cd_h8, a), __builtin_bit_cast(cd_h8, b), c, 0, 0, 0);
}
template <int DT>
__device__ __forceinline__ uint32_t cd_pack(float lo, float hi) {
    const cd_f2 v = {lo, hi};
    if constexpr (DT == BF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, cd_b2));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, cd_h2));
}
template <int DT>
__device__ __forceinline__ uint16_t cd_round(float v) { return DT == BF16 ? f32_to_bf16(v) : f32_to_f16(v); }
template <int DT>
__device__ __forceinline__ float cd_value(uint16_t v) { return DT == BF16 ? bf16_to_f32(v) : f16_to_f32(v); }
template <int DT>
__device__ __forceinline__ float2 cd_unpack(uint32_t w) {
    return make_float2(cd_value<DT>((uint16_t)w), cd_value<DT>((uint16_t)(w >> 16)));
}

// Eight consecutive 16-bit elements from an odd or even start: five dwords
// from the one below, shifted by sh = 0 or 16 bits.
__device__ __forceinline__ uint4 cd_frag(const uint32_t *s, uint32_t sh) {
    const uint32_t q0 = s[0], q1 = s[1], q2 = s[2], q3 = s[3], q4 = s[4];
    return make_uint4(__builtin_amdgcn_alignbit(q1, q0, sh), __builtin_amdgcn_alignbit(q2, q1, sh),
                      __builtin_amdgcn_alignbit(q3, q2, sh), __builtin_amdgcn_alignbit(q4, q3, sh));
}

// Exponent that puts max |k_t| (skip added to tap 0) of a kernel row into
// [2^14, 2^15), over the whole workgroup; red: one float per wave.  A barrier
// separates the call from the last use of red.
__device__ __forceinline__ int cd_kernel_exp(const float *k, int n, float skip, float *red, int tid, int nt) {
    float mx = 0.f;
    for (int t = tid; t < n; t += nt) mx = fmaxf(mx, fabsf(t == 0 ? k[0] + skip : k[t]));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    for (int v = 0; v < nt >> 6; ++v) mx = fmaxf(mx, red[v]);
    return pow2_exp(mx) - 15;
}

// v = hi + lo in 16 bits
template <int DT>
__device__ __forceinline__ void cd_split(float v, uint16_t &hi, uint16_t &lo) {
    hi = cd_round<DT>(v);
    lo = cd_round<DT>(v - cd_value<DT>(hi));
}

}  // namespace h3
