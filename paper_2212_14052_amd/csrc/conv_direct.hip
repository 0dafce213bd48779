// Fused convolution of 16-bit rows by direct summation on the matrix cores
// (L = 256, 512 and 1024; L = 2048 and 8192 up have their own transforms, other
// lengths and float32 the VALU transform):
//     y[t] = sum_{s <= t} k[t-s] u[s] + D u[t],
// or, for the input gradient, the correlation sum_{s >= t} k[s-t] u[s] + D u[t].
//
// u enters as fp16, bf16 rows scaled by a power of two; the float32 kernel
// (skip term in its first tap), scaled likewise, is split into two fp16
// pieces, k = hi + lo, so that every product is exact in the matrix core's
// float32 and the result is the float32 sum of a kernel off by 2^-23 at most,
// where a float32 transform rounds at every pass.  (A kernel of cancelling taps,
// rms 1.15, at L = 1024 came out 3.7e-6 off, by the float32 transform 1.0e-5; with
// the kernel in bf16 pieces, 2^-17, it was 1.7e-4.)
//
// One tile product, rows i < 16, columns n < 16, reduction kk < 32:
//     D[i][n] += sum_kk A[i][kk] B[kk][n],   A[i][kk] = k[tau + 16 + i - kk],
//                                            B[kk][n] = u[t0 + 16 n - tau - 16 + kk]
// adds the lags tau + 16 + i - kk to y[t0 + 16 n + i].  With tau = 256 d + rho
// the kernel tiles A_d and the input tiles B_a (at 256 a - rho) form a
// product of polynomials over 256-blocks, D_b += sum_d A_d B_{b-d}, so NB
// tiles of each feed NB (NB + 1) / 2 products (NB = L / 256) and the half
// square above the diagonal is left out.
//
// Split of the work: one wave per R rows of a channel, all waves of a
// workgroup on one channel, whose kernel pieces they share in LDS (read as
// five dwords and shifted by half a dword where a lane's taps start at an odd
// element).  R = 2 reads each kernel tile once for two rows (B = 8, H = 768, L =
// 1024: R = 1 / 2 / 4: 29 / 27 / 30 us with the kernel generation).  Bound by
// the matrix cores, L^2 (1 + 256 / L) multiply-adds per row, and by the LDS
// reads.  The work grows with L^2: at L = 4096 one row per wave took 134 us at B
// = 5, H = 767, where the transform takes 87.
//
// Measured, with the kernel generation, float32 transform -> this (us): B = 8,
// H = 768, L = 1024: fp16 29.4 -> 23.3, bf16 31.0 -> 23.2; B = 16, H = 2048: 97 -> 83,
// 102 -> 84; B = 1, H = 4096: 51 -> 43, 53 -> 43; L = 512, B = 8, H = 768, bf16: 19.1
// -> 18.2.  Level where the two calls' host time covers it, from L = 256 to B = 1, H =
// 768 at 1024; B = 2, H = 1500 at 1024, one wave per workgroup: 24.9 -> 26.0, 25.6 -> 26.3.
#include "direct_conv.h"
#include "internal.h"

namespace h3 {
namespace {

constexpr int CD_MAXW = 8;

// LDS elements (16-bit) of the two kernel pieces and of a row slot
template <int NB>
struct CdPlan {
    static constexpr int L = 256 * NB;
    static constexpr int KS = L + 24, US = L + 240;
    static constexpr size_t lds(int waves, int R) { return 2 * (2 * (size_t)KS + (size_t)waves * R * US); }
};

// Workgroup: one channel, `blockDim.x / 64` waves of R rows each.  CONJ: the
// correlation y[t] = sum_{s>=t} k[s-t] u[s] (+ D u[t]) instead.  HEADS: the rows
// are the outer products u_i v_j of the layer with heads of 2^lg channels,
// formed on the way into LDS instead of by a kernel of their own through
// memory (the whole layer at L = 1024, us: B = 4, d = 1280, d_h = 8, bf16: 220 ->
// 205; B = 6, d = 1280, d_h = 8, fp16: 300 -> 280; B = 1, d = 256, d_h = 2: 39 -> 36).
template <int DT, int NB, int R, bool CONJ, bool HEADS>
__global__ __launch_bounds__(64 * CD_MAXW, 4) void conv_direct_kernel(const uint16_t *u, const float *k, const float *D,
                                                                     uint16_t *y, int B, int H, int wg_per_ch,
                                                                     const uint16_t *v, int lg) {
    using P = CdPlan<NB>;
    constexpr int L = P::L;
    extern __shared__ __attribute__((aligned(16))) uint16_t cd_sm[];
    __shared__ float red[CD_MAXW];
    const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x, nw = nt >> 6;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // HEADS: a head's channels on one XCD, whose L2 then serves their shared rows
    const int blk = HEADS ? xcd_logical_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const int h = blk / wg_per_ch, part = blk % wg_per_ch;
    const int i16 = lane & 15, g = lane >> 4;
    const int b0 = (part * nw + w) * R, nr = min(R, B - b0);   // may be <= 0
    uint16_t *kh = cd_sm, *kl = cd_sm + P::KS;
    uint16_t *us = cd_sm + 2 * P::KS + w * R * P::US;

    // the channel's kernel, then the wave's rows: every load in flight at once
    CdKernel<L> kr;
    kr.load(k + (long)h * L, D ? D[h] : 0.f, tid, nt);
    // the wave's rows into LDS, zeros in front (behind, for the correlation)
    constexpr int PIECES = L / 8, PT = (PIECES + 63) / 64;
    cd_u4 raw[R][PT], rav[HEADS ? R : 1][PT];
    const int ku = HEADS ? h >> lg : h, kv = ((h >> (2 * lg)) << lg) + (h & ((1 << lg) - 1)), Hu = HEADS ? H >> lg : H;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            // (rows and pieces past the end: the last one again, never used)
            const long row = (long)min(b0 + r, B - 1) * Hu;
            const int piece = 8 * min(64 * p + lane, PIECES - 1);
            raw[r][p] = *(const cd_u4 *)(u + (row + ku) * L + piece);
            if constexpr (HEADS) rav[r][p] = *(const cd_u4 *)(v + (row + kv) * L + piece);
        }

    // the kernel as two fp16 pieces hi + lo, times a power of two that puts its
    // largest value in [2^14, 2^15), so that lo stays normal, reversed: element
    // L - t holds k_t (the correlation: element 16 + t)
    const int ek = cd_group_exp(kr.max_abs(), red, tid, nt);
#pragma unroll
    for (int i = 0; i < CdKernel<L>::N; ++i) {
        const int t = tid + i * nt, x = CONJ ? 16 + t : L - t;
        if (i * nt < L && t < L) cd_split(ldexpf(kr.v[i], -ek), kh[x], kl[x]);
    }
    // zeros: lags below 0 and (reversed: element 0) from L on
    for (int x = tid; x < 24; x += nt) {
        const int z = CONJ ? (x < 16 ? x : L + x) : (x == 0 ? 0 : L + x);
        kh[z] = 0;
        kl[z] = 0;
    }
    int er[R];   // the rows' exponents
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint16_t *ur = us + r * P::US;
        if constexpr (HEADS) {
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const cd_u4 x = raw[r][p], z = rav[r][p];
                raw[r][p] = cd_u4{mul_16x2<DT>(x[0], z[0]), mul_16x2<DT>(x[1], z[1]), mul_16x2<DT>(x[2], z[2]), mul_16x2<DT>(x[3], z[3])};
            }
        }
        er[r] = ek;
        if constexpr (DT == BF16) er[r] += cd_bf16_to_f16(raw[r]);
#pragma unroll
        for (int p = 0; p < PT; ++p) *(cd_u4 *)(ur + (CONJ ? 0 : 240) + 8 * min(64 * p + lane, PIECES - 1)) = raw[r][p];
        if (lane < 30) *(uint4 *)(ur + (CONJ ? L : 0) + 8 * lane) = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    if (nr <= 0) return;   // whole waves; no barrier follows

    cd_f4 acc[R][NB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[r][b] = cd_f4{0.f, 0.f, 0.f, 0.f};
    // A: lags 256 d + rho + 16 + i - kk (correlation: 256 d + rho + kk - i),
    // kk = 8 g + e; five dwords from the even element below, shifted
    const int e0 = CONJ ? 16 - i16 + 8 * g : L - 16 - i16 + 8 * g;
    const uint32_t sh = (uint32_t)(i16 & 1) * 16;
    const uint32_t *kh32 = (const uint32_t *)kh + (e0 >> 1), *kl32 = (const uint32_t *)kl + (e0 >> 1);
    // B: inputs 256 a - rho - 16 + 16 n + kk (correlation: 256 a + rho + 16 n + kk)
    const uint16_t *ub = us + (CONJ ? 0 : 224) + 16 * i16 + 8 * g;
#pragma unroll 1
    for (int rho = 0; rho < 256; rho += 32) {
        uint4 Ah[NB], Al[NB];
#pragma unroll
        for (int d = 0; d < NB; ++d) {
            const int o = (CONJ ? rho : -rho) / 2 + (CONJ ? 128 : -128) * d;
            Ah[d] = cd_frag(kh32 + o, sh);
            Al[d] = cd_frag(kl32 + o, sh);
        }
#pragma unroll
        for (int a = 0; a < NB; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (r > 0 && r >= nr) continue;
                const uint4 Bv = *(const uint4 *)(ub + r * P::US + 256 * a + (CONJ ? rho : -rho));
#pragma unroll
                for (int d = 0; d < NB; ++d) {
                    const int b = CONJ ? a - d : a + d;
                    if (b >= 0 && b < NB) acc[r][b] = cd_mfma(Ah[d], Bv, acc[r][b]);
                }
#pragma unroll
                for (int d = 0; d < NB; ++d) {
                    const int b = CONJ ? a - d : a + d;
                    if (b >= 0 && b < NB) acc[r][b] = cd_mfma(Al[d], Bv, acc[r][b]);
                }
            }
    }
    // (the exponent applied to each value: 2^er alone may leave float32)
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r < nr) {
            uint16_t *yr = y + ((long)(b0 + r) * H + h) * L + 16 * i16 + 4 * g;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                *(uint2 *)(yr + 256 * b) = make_uint2(pack_16x2<DT>(ldexpf(acc[r][b][0], er[r]), ldexpf(acc[r][b][1], er[r])),
                                                      pack_16x2<DT>(ldexpf(acc[r][b][2], er[r]), ldexpf(acc[r][b][3], er[r])));
        }
}

template <int DT, int NB, int R, bool CONJ, bool HEADS>
hipError_t launch_direct_h(const ConvArgs &a, const float *k, hipStream_t s) {
    using P = CdPlan<NB>;
    const int groups = (a.B + R - 1) / R;
    int wgc = (groups + CD_MAXW - 1) / CD_MAXW;
    while ((long)a.H * wgc < 512 && wgc * 2 <= groups) wgc *= 2;
    const int nw = (groups + wgc - 1) / wgc;
    static_assert(P::lds(CD_MAXW, R) <= 65536 - 1024, "no larger dynamic LDS asked for");
    const size_t lds = P::lds(nw, R);
    hipLaunchKernelGGL((conv_direct_kernel<DT, NB, R, CONJ, HEADS>), dim3((unsigned)(a.H * wgc)), dim3(64 * nw), lds, s, (const uint16_t *)a.u, k, a.D,
                       (uint16_t *)a.y, a.B, a.H, wgc, (const uint16_t *)a.heads_v, a.heads_log2);
    return hipGetLastError();
}

template <int DT, int NB, int R, bool CONJ>
hipError_t launch_direct(const ConvArgs &a, const float *k, hipStream_t s) {
    if constexpr (!CONJ)
        if (a.heads_v) return launch_direct_h<DT, NB, R, false, true>(a, k, s);
    return launch_direct_h<DT, NB, R, CONJ, false>(a, k, s);
}

template <int DT, bool CONJ>
hipError_t launch_direct_nb(const ConvArgs &a, const float *k, hipStream_t s) {
    switch (a.L) {
        case 256: return a.B >= 2 ? launch_direct<DT, 1, 2, CONJ>(a, k, s) : launch_direct<DT, 1, 1, CONJ>(a, k, s);
        case 512: return a.B >= 2 ? launch_direct<DT, 2, 2, CONJ>(a, k, s) : launch_direct<DT, 2, 1, CONJ>(a, k, s);
        case 1024: return a.B >= 2 ? launch_direct<DT, 4, 2, CONJ>(a, k, s) : launch_direct<DT, 4, 1, CONJ>(a, k, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool conv_direct_supported(int L, int dtype) {
    return (dtype == F16 || dtype == BF16) && (L == 256 || L == 512 || L == 1024);
}

hipError_t launch_conv_direct(const ConvArgs &a, const float *k, hipStream_t s) {
    if (!conv_direct_supported(a.L, a.dtype) || a.pair_mode != 0 || a.corr || a.gate || (a.heads_v && a.conj_k)) return hipErrorInvalidValue;
    if (a.dtype == F16) return a.conj_k ? launch_direct_nb<F16, true>(a, k, s) : launch_direct_nb<F16, false>(a, k, s);
    return a.conj_k ? launch_direct_nb<BF16, true>(a, k, s) : launch_direct_nb<BF16, false>(a, k, s);
}

}  // namespace h3
