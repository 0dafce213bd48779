// Shared by the kernels that convolve or correlate 16-bit rows by direct summation on the
// matrix cores: 16x16x32 products, 16-bit pairs, bf16 rows as scaled fp16, and
// operands whose elements start at any 16-bit offset of an LDS array.
#pragma once
#include "common.h"

namespace h3 {

typedef _Float16 cd_h8 __attribute__((ext_vector_type(8)));
typedef unsigned cd_u4 __attribute__((ext_vector_type(4)));
typedef float cd_f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ cd_f4 cd_mfma(uint4 a, uint4 b, cd_f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(cd_h8, a), __builtin_bit_cast(cd_h8, b), c, 0, 0, 0);
}
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

// Exponent that puts the largest of the workgroup's values, mx of each thread
// (not below 0), into [2^14, 2^15); red: one float per wave (nt = 64: the
// wave's own, without barrier).  A barrier separates the call from the last use
// of red.
__device__ __forceinline__ int cd_group_exp(float mx, float *red, int tid, int nt) {
    mx = __uint_as_float(group_max<64>(__float_as_uint(mx)));   // (bits order floats >= 0)
    if (nt > 64) {
        if ((tid & 63) == 0) red[tid >> 6] = mx;
        __syncthreads();
        for (int v = 0; v < nt >> 6; ++v) mx = fmaxf(mx, red[v]);
    }
    return pow2_exp(mx) - 15;
}

// A kernel row's L values over nt threads, the skip weight added to tap 0:
// thread tid holds t = tid + i nt.
template <int L>
struct CdKernel {
    static constexpr int N = L / 64;
    float v[N];
    __device__ __forceinline__ void load(const float *k, float skip, int tid, int nt) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            v[i] = 0.f;
            if (i * nt < L && tid + i * nt < L) v[i] = k[tid + i * nt];
        }
        if (tid == 0) v[0] += skip;
    }
    __device__ __forceinline__ float max_abs() const {
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < N; ++i) mx = fmaxf(mx, fabsf(v[i]));
        return mx;
    }
};

// v = hi + lo in fp16: |v - hi - lo| <= 2^-23 |v| (half a unit of lo, which is
// below half a unit of hi), where lo is a normal number
__device__ __forceinline__ void cd_split(float v, uint16_t &hi, uint16_t &lo) {
    hi = f32_to_f16(v);
    lo = f32_to_f16(v - f16_to_f32(hi));
}

// A row of bf16 values, 16 bytes per lane and piece, as fp16 times a power of
// two: exact down to 2^-29 of its largest value (bf16's 8 bits in fp16's 11,
// subnormals from there), so that it can meet fp16 pairs.  The returned
// exponent e puts the largest value into [2^14, 2^15) (value = fp16 2^e); a
// row that holds an infinity or NaN becomes NaN throughout.
template <int P>
__device__ __forceinline__ int cd_bf16_to_f16(cd_u4 (&x)[P]) {
    typedef unsigned short u2 __attribute__((ext_vector_type(2)));
    u2 m = {0, 0};
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u2, x[p][i] & 0x7fff7fffu));
    const int mx = __builtin_amdgcn_readfirstlane((int)group_max<64>(max(m.x, m.y)));
    const int e = (mx >> 7) - 126 - 15;   // frexp's exponent, from the bits
    const bool finite = mx < 0x7f80;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float2 v = cd_unpack<BF16>(x[p][i]);
            x[p][i] = finite ? pack_16x2<F16>(ldexpf(v.x, -e), ldexpf(v.y, -e)) : 0x7e007e00u;
        }
    return e;
}

}  // namespace h3
