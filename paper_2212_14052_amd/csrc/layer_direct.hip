// The sequence mixing of the H3 layer (Sec. 3.2, Algorithm 1, head dimension
// 1) for rows of 256, 512 and 1024, in one kernel on the matrix cores:
//     Kbar = shift FIR of K (+ shift_D K),  G = Kbar V,
//     O = Q (diag_k (*) G + diag_D G),
// on (B, d, L) rows, O channel-major.
//
// Both convolutions are direct sums (see the direct convolution kernel for the
// tile product) of fp16 operands, each row, kernel and tap set scaled by a power
// of two: the FIR's 64 float32 taps as a pair against K (bf16 fits), three tiles
// per 256 outputs; the diagonal SSM's kernel as a pair against G as a pair, k_hi
// G_hi + k_lo G_hi + k_hi G_lo.  A pair is off by 2^-23 at most and the product
// left out is below 2^-22 of its term.  With cancelling parameters (L = 1024) the
// second sum comes out 3.1e-6 off, where the float32 transform before was 3.6e-6
// off, and the first 1.3e-6 (float32 multiply-adds 0.6e-6; bf16 pieces of the taps
// 6e-5).  G is a float32 value between the two; nothing of it reaches memory.
//
// One wave carries R rows of a channel through all steps; K, then G_hi and
// G_lo lie in the wave's own LDS slots, so that after the channel's kernel and
// taps are in LDS no barrier is needed.  V and Q are read, and O is written,
// where a lane's four consecutive results of a tile lie.  Bound by the matrix
// cores (about 4200 cycles per row at L = 1024) and the LDS reads beside them.
//
// B = 8, d = 768, L = 1024, fp16: 27 us, against 101 us for the float32
// transform in LDS, 6.5 for its kernel spectra and 7 for the transpose that
// its result went through.
#include "direct_conv.h"
#include "internal.h"

namespace h3 {
namespace {

constexpr int LD_MAXW = 8;
constexpr int LD_TAPS = 128;   // LDS elements per tap piece: lags 95 .. -16, reversed

template <int NB>
struct LdPlan {
    static constexpr int L = 256 * NB;
    static constexpr int KS = L + 24, GS = L + 240;   // elements of a kernel piece, of a G piece
    static constexpr size_t lds(int waves, int R) {
        return 2 * (2 * (size_t)KS + 2 * LD_TAPS + (size_t)waves * R * 2 * GS);
    }
};

template <int DT, int NB, int R>
__global__ __launch_bounds__(64 * LD_MAXW, 2) void layer_direct_kernel(const uint16_t *q, const uint16_t *k,
                                                                      const uint16_t *v, const float *shift_C,
                                                                      const float *shift_D, int m_s, const float *diag_k,
                                                                      const float *diag_D, int B, int d, int wg_per_ch,
                                                                      uint16_t *o) {
    using P = LdPlan<NB>;
    constexpr int L = P::L;
    extern __shared__ __attribute__((aligned(16))) uint16_t ld_sm[];
    __shared__ float red[LD_MAXW];
    const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x, nw = nt >> 6;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = blockIdx.x / wg_per_ch, part = blockIdx.x % wg_per_ch;
    const int i16 = lane & 15, g = lane >> 4;
    const int b0 = (part * nw + w) * R, nr = min(R, B - b0);   // may be <= 0
    uint16_t *kh = ld_sm, *kl = kh + P::KS, *th = kl + P::KS, *tl = th + LD_TAPS;
    uint16_t *slot = tl + LD_TAPS + w * R * 2 * P::GS;

    // the channel's kernel, and its taps, one per lane of every wave
    CdKernel<L> kr;
    kr.load(diag_k + (long)c * L, diag_D ? diag_D[c] : 0.f, tid, nt);
    float tap = lane < m_s ? shift_C[(long)c * m_s + lane] : 0.f;
    if (lane == 0 && shift_D) tap += shift_D[c];
    // K of the wave's rows (rows past the end: the last one again, never used)
    constexpr int PIECES = L / 8, PT = (PIECES + 63) / 64;
    cd_u4 raw[R][PT];
    long ro[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        ro[r] = ((long)min(b0 + r, B - 1) * d + c) * L;
#pragma unroll
        for (int p = 0; p < PT; ++p) raw[r][p] = *(const cd_u4 *)(k + ro[r] + 8 * min(64 * p + lane, PIECES - 1));
    }
    // the lane's V: outputs 256 b + 16 i16 + 4 g .. + 3
    const int lo4 = 16 * i16 + 4 * g;
    uint2 vv[R][NB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) vv[r][b] = *(const uint2 *)(v + ro[r] + 256 * b + lo4);

    // diag_k as an fp16 pair, reversed: element L - t holds tap t
    const int ek = cd_group_exp(kr.max_abs(), red, tid, nt);
#pragma unroll
    for (int i = 0; i < CdKernel<L>::N; ++i) {
        const int t = tid + i * nt;
        if (i * nt < L && t < L) cd_split(ldexpf(kr.v[i], -ek), kh[L - t], kl[L - t]);
    }
    for (int x = tid; x < 24; x += nt) {
        const int z = x == 0 ? 0 : L + x;
        kh[z] = 0;
        kl[z] = 0;
    }
    // the shift taps as an fp16 pair, reversed: element 96 - j holds tap j
    const int et = cd_group_exp(fabsf(tap), red, lane, 64);   // (64: the wave's own maximum)
    if (w == 0) {
        cd_split(ldexpf(tap, -et), th[96 - lane], tl[96 - lane]);
        const int z = lane < 33 ? lane : 64 + lane;   // 0 .. 32, 97 .. 127
        th[z] = 0;
        tl[z] = 0;
    }
    // K behind 80 zeros, in the row's first piece
    int eb[R];   // the exponents of the rows' Kbar
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint16_t *s = slot + r * 2 * P::GS;
        eb[r] = et;
        if constexpr (DT == BF16) eb[r] += cd_bf16_to_f16(raw[r]);
#pragma unroll
        for (int p = 0; p < PT; ++p) *(cd_u4 *)(s + 80 + 8 * min(64 * p + lane, PIECES - 1)) = raw[r][p];
        if (lane < 10) *(uint4 *)(s + 8 * lane) = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    if (nr <= 0) return;   // whole waves; no barrier follows

    // ---- Kbar, then G = Kbar V ----
    cd_f4 acc[R][NB];
    {
        // A: lags tau + 16 + i - kk, tau = 0, 32, 64;  B: K[256 b + 16 n - tau - 16 + kk]
        const int e0 = 96 - 16 - i16 + 8 * g;
        const uint32_t sh = (uint32_t)(e0 & 1) * 16;
        uint4 Th[3], Tl[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            Th[p] = cd_frag((const uint32_t *)th + (e0 >> 1) - 16 * p, sh);
            Tl[p] = cd_frag((const uint32_t *)tl + (e0 >> 1) - 16 * p, sh);
        }
        const uint16_t *kb = slot + 80 - 16 + 16 * i16 + 8 * g;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                cd_f4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const uint4 Bv = *(const uint4 *)(kb + r * 2 * P::GS + 256 * b - 32 * p);
                    s = cd_mfma(Th[p], Bv, s);
                    s = cd_mfma(Tl[p], Bv, s);
                }
                acc[r][b] = s;
            }
    }
    int eg[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float mx = 0.f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float2 v0 = cd_unpack<DT>(vv[r][b].x), v1 = cd_unpack<DT>(vv[r][b].y);
            acc[r][b][0] = ldexpf(acc[r][b][0], eb[r]) * v0.x;
            acc[r][b][1] = ldexpf(acc[r][b][1], eb[r]) * v0.y;
            acc[r][b][2] = ldexpf(acc[r][b][2], eb[r]) * v1.x;
            acc[r][b][3] = ldexpf(acc[r][b][3], eb[r]) * v1.y;
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = fmaxf(mx, fabsf(acc[r][b][e]));
        }
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) mx = fmaxf(mx, __shfl_xor(mx, s, 64));
        eg[r] = __builtin_amdgcn_readfirstlane(pow2_exp(mx)) - 15;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();   // the wave's reads of K are done before G takes its place
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint16_t *gh = slot + r * 2 * P::GS, *gl = gh + P::GS;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float x[4], y[4];
            // (the exponent applied to each value, here and below: the power of
            // two alone leaves float32 for rows below 2^-113)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = ldexpf(acc[r][b][e], -eg[r]);
            const uint2 hi = make_uint2(pack_16x2<F16>(x[0], x[1]), pack_16x2<F16>(x[2], x[3]));
            const float2 h0 = cd_unpack<F16>(hi.x), h1 = cd_unpack<F16>(hi.y);
            y[0] = x[0] - h0.x; y[1] = x[1] - h0.y; y[2] = x[2] - h1.x; y[3] = x[3] - h1.y;
            *(uint2 *)(gh + 240 + 256 * b + lo4) = hi;
            *(uint2 *)(gl + 240 + 256 * b + lo4) = make_uint2(pack_16x2<F16>(y[0], y[1]), pack_16x2<F16>(y[2], y[3]));
        }
        if (lane < 30) {
            *(uint4 *)(gh + 8 * lane) = make_uint4(0, 0, 0, 0);
            *(uint4 *)(gl + 8 * lane) = make_uint4(0, 0, 0, 0);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    // ---- S = diag_k (*) G ----
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            acc[r][b] = cd_f4{0.f, 0.f, 0.f, 0.f};
            vv[r][b] = *(const uint2 *)(q + ro[r] + 256 * b + lo4);   // Q
        }
    const int e0 = L - 16 - i16 + 8 * g;
    const uint32_t sh = (uint32_t)(e0 & 1) * 16;
    const uint32_t *kh32 = (const uint32_t *)kh + (e0 >> 1), *kl32 = (const uint32_t *)kl + (e0 >> 1);
    const uint16_t *gb = slot + 224 + 16 * i16 + 8 * g;
#pragma unroll 1
    for (int rho = 0; rho < 256; rho += 32) {
        uint4 Ah[NB], Al[NB];
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            Ah[e] = cd_frag(kh32 - rho / 2 - 128 * e, sh);
            Al[e] = cd_frag(kl32 - rho / 2 - 128 * e, sh);
        }
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint4 Bh = *(const uint4 *)(gb + r * 2 * P::GS + 256 * a - rho);
                const uint4 Bl = *(const uint4 *)(gb + r * 2 * P::GS + P::GS + 256 * a - rho);
#pragma unroll
                for (int e = 0; a + e < NB; ++e) acc[r][a + e] = cd_mfma(Ah[e], Bh, acc[r][a + e]);
#pragma unroll
                for (int e = 0; a + e < NB; ++e) acc[r][a + e] = cd_mfma(Al[e], Bh, acc[r][a + e]);
#pragma unroll
                for (int e = 0; a + e < NB; ++e) acc[r][a + e] = cd_mfma(Ah[e], Bl, acc[r][a + e]);
            }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r >= nr) continue;
        const int eo = ek + eg[r];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float2 q0 = cd_unpack<DT>(vv[r][b].x), q1 = cd_unpack<DT>(vv[r][b].y);
            *(uint2 *)(o + ro[r] + 256 * b + lo4) =
                make_uint2(pack_16x2<DT>(ldexpf(acc[r][b][0], eo) * q0.x, ldexpf(acc[r][b][1], eo) * q0.y),
                           pack_16x2<DT>(ldexpf(acc[r][b][2], eo) * q1.x, ldexpf(acc[r][b][3], eo) * q1.y));
        }
    }
}

template <int DT, int NB, int R>
hipError_t launch_ld(const void *q, const void *k, const void *v, const float *shift_C, const float *shift_D, int m_s,
                     const float *diag_k, const float *diag_D, int B, int d, void *o, hipStream_t s) {
    const int groups = (B + R - 1) / R;
    int wgc = (groups + LD_MAXW - 1) / LD_MAXW;
    while ((long)d * wgc < 512 && wgc * 2 <= groups) wgc *= 2;
    const int nw = (groups + wgc - 1) / wgc;
    const size_t lds = LdPlan<NB>::lds(nw, R);
    auto fn = layer_direct_kernel<DT, NB, R>;
    if (lds > 60000) (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(fn, dim3((unsigned)(d * wgc)), dim3(64 * nw), lds, s, (const uint16_t *)q, (const uint16_t *)k,
                       (const uint16_t *)v, shift_C, shift_D, m_s, diag_k, diag_D, B, d, wgc, (uint16_t *)o);
    return hipGetLastError();
}

template <int DT>
hipError_t launch_ld_dt(const void *q, const void *k, const void *v, const float *shift_C, const float *shift_D,
                        int m_s, const float *diag_k, const float *diag_D, int B, int d, int L, void *o,
                        hipStream_t s) {
#define H3_LD(NB)                                                                                               \
    return B >= 2 ? launch_ld<DT, NB, 2>(q, k, v, shift_C, shift_D, m_s, diag_k, diag_D, B, d, o, s)            \
                  : launch_ld<DT, NB, 1>(q, k, v, shift_C, shift_D, m_s, diag_k, diag_D, B, d, o, s)
    switch (L) {
        case 256: H3_LD(1);
        case 512: H3_LD(2);
        case 1024: H3_LD(4);
    }
#undef H3_LD
    return hipErrorInvalidValue;
}

}  // namespace

bool layer_direct_supported(int L) { return L == 256 || L == 512 || L == 1024; }

hipError_t launch_layer_direct(const void *q, const void *k, const void *v, const float *shift_C, const float *shift_D,
                               int m_s, const float *diag_k, const float *diag_D, int B, int d, int L, int dtype,
                               void *o, hipStream_t s) {
    if (m_s > 64) return hipErrorInvalidValue;
    return dtype == BF16 ? launch_ld_dt<BF16>(q, k, v, shift_C, shift_D, m_s, diag_k, diag_D, B, d, L, o, s)
                         : launch_ld_dt<F16>(q, k, v, shift_C, shift_D, m_s, diag_k, diag_D, B, d, L, o, s);
}

}  // namespace h3
