// State passing (Sec. 4.2, Algorithm 2) for 16-bit rows in one pass over the
// sequence, on the matrix cores.
//
// The state-passing identity holds for any chunk length (Proposition 2), so
// the kernel picks its own: blocks of Q = 64 inputs.  With T the 64 x 64
// Toeplitz matrix of the first taps (skip term included) and x_n the state
// before block n,
//     y_n = T u_n + M_xy x_n,      x_{n+1} = Abar^Q x_n + M_ux u_n.
// A wave walks a row (or a segment of it) 32 blocks at a time.  The three
// products are 32x32x16 matrix instructions with the 32 blocks as columns: per
// input about 40 + 128 + 128 multiply-adds, against the transforms of a
// chunked FFT convolution and a separate pass for the chunk states.
//   M_ux u    the blocks' end states from zero (rows = blocks, column = mode);
//             one swap of the wave's halves per register makes lane = mode
//             with all 32 blocks in the lane's registers, so that
//   the scan  is 32 complex multiply-adds per lane in float32, with no
//             cross-lane step;
//   M_xy x    the states, scaled by a common power of two to fp16, change from
//             lane = mode to lane = block through LDS (8.5 KB per wave).
// Inputs and outputs pass through the same LDS buffer so that memory is read
// and written in whole lines; the stores are non-temporal (a copy with this
// pattern: 5.2 TB/s, 4.0 with ordinary stores; the fragments' own 32-byte
// pieces reach 2.1).  Tables: M_ux and T in registers, M_xy in LDS, shared by
// the workgroup's waves.
//
// Precision: M_ux and T in 16 bits for fp16 rows, as 16-bit hi + lo pairs for
// bf16 rows (two products); M_xy and the scaled states in fp16; the state and
// its decay over blocks in float32 from float64 powers, what a step's 32 factors
// miss of theirs added back.  theta scales each
// mode so that its tables have moduli just below 1, where fp16 rounds finest.
//
// Bound by the serial chain of each wave at two waves per SIMD (about 440 VALU
// and 38 matrix instructions per 2048 inputs): B = 2, H = 1024, L = 131072, fp16:
// 270-280 us = 3.9 TB/s (305 us on a slower card, where the same loop without the
// arithmetic took 257); chunk states and convolution before: 708 us.
#include "common.h"
#include "internal.h"

namespace h3 {
namespace {

typedef _Float16 sc_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 sc_h2 __attribute__((ext_vector_type(2)));
typedef __bf16 sc_b8 __attribute__((ext_vector_type(8)));
typedef float sc_f16 __attribute__((ext_vector_type(16)));

constexpr int SC_Q = 64;             // inputs per block
constexpr int SC_STEP = 32 * SC_Q;   // inputs per step: 32 blocks, the columns of a tile
constexpr int SC_PITCH = 68;         // words per block in the state exchange
constexpr int SC_UP = 144;           // bytes per block in the input and output exchange
constexpr int SC_XB = 32 * SC_PITCH * 4;   // bytes of a wave's exchange buffer
static_assert(32 * SC_UP <= SC_XB, "the exchanges share a buffer");

// acc + A B: rows i < 32, columns n < 32, reduction k < 16; lane c + 32 g holds
// A[c][8 g ..], B[8 g ..][c] and of the result rows 8 (r / 4) + 4 g + r % 4 of column c
template <int DT>
__device__ __forceinline__ sc_f16 sc_mfma(uint4 a, uint4 b, sc_f16 c) {
    if constexpr (DT == BF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sc_b8, a), __builtin_bit_cast(sc_b8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(sc_h8, a), __builtin_bit_cast(sc_h8, b), c, 0, 0, 0);
}
template <int DT>
__device__ __forceinline__ float2 sc_unpack(uint32_t w) {
    if constexpr (DT == BF16) return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u));
    const sc_h2 h = __builtin_bit_cast(sc_h2, w);
    return make_float2((float)h.x, (float)h.y);
}
// eight floats as a 16-bit operand and, in lo, what the rounding left over
template <int DT>
__device__ __forceinline__ uint4 sc_pack8(const float (&v)[8], uint4 *lo) {
    uint32_t hi[4], lw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        hi[i] = pack_16x2<DT>(v[2 * i], v[2 * i + 1]);
        const float2 r = sc_unpack<DT>(hi[i]);
        lw[i] = pack_16x2<DT>(v[2 * i] - r.x, v[2 * i + 1] - r.y);
    }
    if (lo) *lo = make_uint4(lw[0], lw[1], lw[2], lw[3]);
    return make_uint4(hi[0], hi[1], hi[2], hi[3]);
}
__device__ __forceinline__ double2 sc_zmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 sc_zpow(double2 z, int e) {
    double2 r = make_double2(1.0, 0.0);
    while (e) {
        if (e & 1) r = sc_zmul(r, z);
        z = sc_zmul(z, z);
        e >>= 1;
    }
    return r;
}
template <int N> __device__ __forceinline__ double2 sc_zsqr(double2 z) {   // z^(2^N)
#pragma unroll
    for (int i = 0; i < N; ++i) z = sc_zmul(z, z);
    return z;
}
// rounded to float32, saturating: a growing mode's power must not turn a state
// that is zero into NaN
__device__ __forceinline__ float sc_float(double v) {
    return (float)fmin(fmax(v, -3.4e38), 3.4e38);   // (NaN: inf - inf, saturates too)
}
__device__ __forceinline__ float2 sc_float2(double2 z) { return make_float2(sc_float(z.x), sc_float(z.y)); }
// a x + s
__device__ __forceinline__ float2 sc_cfma(float2 a, float2 x, float2 s) {
    return make_float2(fmaf(a.x, x.x, fmaf(-a.y, x.y, s.x)), fmaf(a.x, x.y, fmaf(a.y, x.x, s.y)));
}
// maximum over the wave, in every lane
template <int N>
__device__ __forceinline__ float sc_ror(float v) {   // rotate within 16 lanes
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float sc_wave_max(float v) {
    v = fmaxf(v, sc_ror<8>(v));
    v = fmaxf(v, sc_ror<4>(v));
    v = fmaxf(v, sc_ror<2>(v));
    v = fmaxf(v, sc_ror<1>(v));
    uint32_t x = __float_as_uint(v);
    const auto s = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    v = fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
    x = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

struct ScanArgs {
    const uint16_t *u;
    uint16_t *y;
    const float *Abar, *Bbar, *C, *D, *x0;
    float *x_final;
    float2 *seg;          // (B, H, nseg, 64) scaled: end states of the segments but the last, then x0
    int B, H, L, m;
    int nseg, seg_steps;  // segments per row, steps per segment
    int items;            // segments per row that this launch runs
    int wg_per_ch;
};

// LDS: the output tables (16 KB), with NP = 2 the low halves of the state
// tables (16 KB), then 8.5 KB per wave for the state exchange.  The set-up's
// scratch lies where the output tables go.
template <int NP, bool STATES>
constexpr size_t scan_lds(int waves) {
    return 16384 * (size_t)NP + SC_XB * (size_t)waves;
}

// NP: 16-bit pieces of the state and Toeplitz tables (1, or 2 for hi + lo).
// STATES: only the segments' end states from a zero state, and x0, to a.seg.
template <int DT, int NP, bool STATES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void ssm_scan_kernel(ScanArgs a) {
    extern __shared__ __attribute__((aligned(16))) char sm[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int c = lane & 31, g = lane >> 5;
    const int h = blockIdx.x / a.wg_per_ch;
    const int item = (blockIdx.x % a.wg_per_ch) * nw + w;

    // ---- set-up: powers of the channel's modes, float32 (scratch) ----
    float2 *P = (float2 *)sm;            // [64][17]: z^(8 t), t < 8, then z^q, q <= 8
    float2 *BW = P + 64 * 17, *CW = BW + 64, *W = CW + 64, *TH = W + 64;
    float *GF = (float *)(TH + 64);
    if (tid < 64) {
        const long i = (long)h * a.m + tid;
        const bool on = tid < a.m;
        const float2 z = on ? make_float2(a.Abar[2 * i], a.Abar[2 * i + 1]) : make_float2(0.f, 0.f);
        const float2 bb = on ? make_float2(a.Bbar[2 * i], a.Bbar[2 * i + 1]) : make_float2(0.f, 0.f);
        const float2 cc = on && !STATES ? make_float2(a.C[2 * i], a.C[2 * i + 1]) : make_float2(0.f, 0.f);
        float2 *p = P + tid * 17;
        float2 q = make_float2(1.f, 0.f);
        for (int t = 0; t <= 8; ++t) {
            p[8 + t] = q;
            if (t < 8) q = cmul(q, z);
        }
        const float2 z8 = q;
        float2 e = make_float2(1.f, 0.f);
        for (int t = 0; t < 8; ++t) {
            p[t] = e;
            e = cmul(e, z8);
        }
        // e = z^64; the table entries' largest moduli, as powers of two
        const float z1 = hypotf(z.x, z.y), z64 = hypotf(e.x, e.y);
        const float2 z63 = cmul(p[7], p[15]);
        // x = theta x': the tables hold moduli just below 1, where the 16-bit
        // rounding is finest (theta no smaller than 2^-60, so that a given
        // initial state stays in range)
        const float zmax = fmaxf(1.f, hypotf(z63.x, z63.y));
        const bool plain = !(hypotf(bb.x, bb.y) * zmax >= 8.7e-19f);
        const float2 th = plain ? make_float2(8.7e-19f, 0.f) : cscale(bb, zmax);
        const float gf = 2.f * hypotf(cc.x, cc.y) * hypotf(th.x, th.y) * fmaxf(z1, z64);
        const float2 ct = cscale(cmul(cc, th), 2.f);
        TH[tid] = th;
        GF[tid] = gf;
        BW[tid] = plain ? cscale(bb, 1.f / 8.7e-19f) : make_float2(1.f / zmax, 0.f);
        CW[tid] = gf > 0.f ? make_float2(ct.x / gf, ct.y / gf) : make_float2(0.f, 0.f);
        W[tid] = cscale(cmul(cc, bb), 2.f);
    }
    __syncthreads();
    // M_ux: mode 32 t + c is the column, input j = 16 k + 8 g + i the
    // reduction: Bbar z^(63 - j) / theta
    uint4 mx[2][2][4], mlo[NP == 2 ? 2 : 1][2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const float2 *p = P + (32 * t + c) * 17;
        const float2 bw = BW[32 * t + c];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float2 pb = cmul(bw, p[7 - 2 * k - g]);
            float re[8], im[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float2 v = cmul(pb, p[8 + 7 - i]);
                re[i] = v.x;
                im[i] = v.y;
            }
            mx[t][0][k] = sc_pack8<DT>(re, NP == 2 ? &mlo[NP == 2 ? t : 0][0][k] : nullptr);
            mx[t][1][k] = sc_pack8<DT>(im, NP == 2 ? &mlo[NP == 2 ? t : 0][1][k] : nullptr);
        }
    }
    const float2 th = TH[lane];
    const float gf = GF[lane];
    const int egf = __builtin_amdgcn_readfirstlane(pow2_exp(sc_wave_max(gf)));   // of the largest
    float *xb = (float *)(sm + 16384 * NP + SC_XB * w);   // the wave's exchange buffer
    // M_xy: row R is output i = 32 rho + 16 (R / 16) + 8 (R / 4 % 2) + 4 (R / 8
    // % 2) + R % 4 (so that a lane ends up with runs of eight consecutive
    // outputs), reduction slot 16 k + 8 g + e: mode 8 k + 4 g + e / 2, e % 2:
    // Re / -Im of 2 C theta z^(i+1) / GF.  Fragment 8 rho + k is built by wave
    // (8 rho + k) % nw.
    const int ri = 16 * (c >> 4) + 8 * ((c >> 2) & 1) + 4 * ((c >> 3) & 1) + (c & 3);
    uint4 fr[STATES ? 1 : 16];
    uint4 tt[STATES ? 1 : 4], tlo[NP == 2 && !STATES ? 4 : 1];
    int eT = 0;
    if constexpr (!STATES) {
#pragma unroll
        for (int f = 0; f < 16; ++f) {
            if (f % nw != w) continue;
            float v[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = 8 * (f & 7) + 4 * g + q, i = 32 * (f >> 3) + ri;
                const float2 *p = P + n * 17;
                const float2 e = cmul(CW[n], cmul(p[i >> 3], p[8 + (i & 7) + 1]));
                v[2 * q] = e.x;
                v[2 * q + 1] = -e.y;
            }
            fr[f] = sc_pack8<F16>(v, nullptr);
        }
        // the kernel's first 64 taps (skip term in tap 0), one per lane
        float kt = lane == 0 && a.D ? a.D[h] : 0.f;
#pragma unroll 8
        for (int n = 0; n < 64; ++n) {
            const float2 *p = P + n * 17;
            const float2 z = cmul(p[lane >> 3], p[8 + (lane & 7)]), wn = W[n];
            kt = fmaf(wn.x, z.x, fmaf(-wn.y, z.y, kt));
        }
        eT = __builtin_amdgcn_readfirstlane(pow2_exp(sc_wave_max(fabsf(kt))));
        xb[lane] = ldexpf(kt, -eT);
        // T: the same rows, reduction j = 8 g + e: taps 16 (d - 1) + i - j
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int t = 16 * (d - 1) + ri - 8 * g - e;
                v[e] = t >= 0 ? xb[t] : 0.f;
            }
            tt[d] = sc_pack8<DT>(v, NP == 2 ? &tlo[NP == 2 ? d : 0] : nullptr);
        }
    }
    __syncthreads();   // every wave has read the scratch
    uint4 *Mxy = (uint4 *)sm, *Mlo = (uint4 *)(sm + 16384);
    if constexpr (!STATES) {
#pragma unroll
        for (int f = 0; f < 16; ++f)
            if (f % nw == w) Mxy[64 * f + lane] = fr[f];
    }
    if constexpr (NP == 2) {
        if (w == 0) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 8; ++q) Mlo[64 * (8 * t + q) + lane] = mlo[t][q >> 2][q & 3];
        }
    }
    __syncthreads();
    if (item >= a.B * a.items) return;   // whole waves; no barrier follows

    // ---- the wave's segment; lane = mode for the states ----
    const int b = item / a.items, sg = item % a.items;
    const long row = (long)b * a.H + h;
    const int nsteps = a.L / SC_STEP;
    const int s0 = sg * a.seg_steps, s1 = min(s0 + a.seg_steps, nsteps);
    const bool on = lane < a.m;
    double2 z = make_double2(0.0, 0.0);
    if (on) z = make_double2(a.Abar[2 * ((long)h * a.m + lane)], a.Abar[2 * ((long)h * a.m + lane) + 1]);
    const double2 z64 = sc_zsqr<6>(z), zstep = sc_zsqr<5>(z64);   // a block's and a step's decay
    static_assert(SC_Q == 64 && SC_STEP == 32 * 64, "powers by squaring");
    const float2 a1 = sc_float2(z64);
    // what 32 factors a1 leave over of a step's z^2048, added once per step: the
    // rounding of a1 would add up (modes that hardly decay, L = 2^18: the state
    // off by 5e-5, with it 2e-6)
    const double2 z32 = sc_zsqr<5>(make_double2((double)a1.x, (double)a1.y));
    const float2 da = sc_float2(make_double2(zstep.x - z32.x, zstep.y - z32.y));
    float2 x = make_float2(0.f, 0.f);
    // the given state.  Of several segments, the launch of the end states alone
    // reads it, and leaves it in the last segment's slot: x_final may be the
    // same buffer, and the last segment's wave writes it while others start
    float2 *const given = a.seg + (row * a.nseg + a.nseg - 1) * 64 + lane;
    if (STATES ? sg == 0 : a.nseg == 1) {
        if (on && a.x0) {
            const long xi = row * a.m + lane;
            const float d = 1.f / fmaf(th.x, th.x, th.y * th.y);
            x = cscale(cmul(make_float2(a.x0[2 * xi], a.x0[2 * xi + 1]), cconj(th)), d);
        }
        if constexpr (STATES) {
            *given = x;
            x = make_float2(0.f, 0.f);
        }
    }
    if constexpr (!STATES) {
        if (a.nseg > 1) x = *given;
        if (sg > 0) {   // the state at the segment's start
            const double2 ps = sc_zpow(zstep, a.seg_steps);
            const float2 as = sc_float2(ps), al = sc_float2(make_double2(ps.x - as.x, ps.y - as.y));
            const float2 *e = a.seg + row * a.nseg * 64 + lane;
#pragma unroll 8
            for (int s = 0; s < sg; ++s) x = sc_cfma(as, x, sc_cfma(al, x, e[64 * s]));
        }
    }

    // a step's 4 KB are read and written in whole lines (lane l: 16 bytes at 16
    // l of each 1 KB) and pass through LDS, block n at SC_UP n, to and from
    // the operand layout (lane c + 32 g: pieces 2 k + g of block c)
    const long off = row * a.L + (long)s0 * SC_STEP + 8 * lane;
    const uint16_t *up = a.u + off;
    uint16_t *yp = a.y + off;
    const uint4 *mxyl = Mxy + lane, *mlol = Mlo + lane;
    uint32_t *xw = (uint32_t *)xb;
    char *const lines = (char *)xb + SC_UP * (lane >> 3) + 16 * (lane & 7);
    char *const frags = (char *)xb + SC_UP * c + 16 * g;
    auto settle = [] {   // one wave: LDS operations stay in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    uint4 n0 = *(const uint4 *)up, n1 = *(const uint4 *)(up + 512), n2 = *(const uint4 *)(up + 1024),
          n3 = *(const uint4 *)(up + 1536);
    const sc_f16 zero = {};
    for (int st = s0; st < s1; ++st) {
        *(uint4 *)lines = n0;
        *(uint4 *)(lines + 8 * SC_UP) = n1;
        *(uint4 *)(lines + 16 * SC_UP) = n2;
        *(uint4 *)(lines + 24 * SC_UP) = n3;
        settle();
        const uint4 u[4] = {*(const uint4 *)frags, *(const uint4 *)(frags + 32), *(const uint4 *)(frags + 64),
                            *(const uint4 *)(frags + 96)};
        settle();
        // the next step's input, one step ahead (the last step reads its own again)
        if (st + 1 < s1) up += SC_STEP;
        n0 = *(const uint4 *)up;
        n1 = *(const uint4 *)(up + 512);
        n2 = *(const uint4 *)(up + 1024);
        n3 = *(const uint4 *)(up + 1536);
        // block end states from a zero state: rows = blocks, column = mode
        sc_f16 sx[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                sx[t][p] = zero;
#pragma unroll
                for (int k = 0; k < 4; ++k) sx[t][p] = sc_mfma<DT>(u[k], mx[t][p][k], sx[t][p]);
                if constexpr (NP == 2) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) sx[t][p] = sc_mfma<DT>(u[k], mlol[64 * (8 * t + 4 * p + k)], sx[t][p]);
                }
            }
        // exchange the halves of the wave between the two mode tiles: lane =
        // mode, and register (r, half) holds block 8 (r / 4) + 4 half + r % 4
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(sx[0][p][r]), __float_as_uint(sx[1][p][r]),
                                                                false, false);
                sx[0][p][r] = __uint_as_float(q[0]);
                sx[1][p][r] = __uint_as_float(q[1]);
            }
        // the states before each block, in place
        float mxv = 0.f;
        const float2 xs = x;
#pragma unroll
        for (int n = 0; n < 32; ++n) {
            const int r = 4 * (n >> 3) + (n & 3), t = (n >> 2) & 1;
            const float2 s = make_float2(sx[t][0][r], sx[t][1][r]);
            if constexpr (!STATES) {
                sx[t][0][r] = x.x;
                sx[t][1][r] = x.y;
                mxv = fmaxf(fmaxf(mxv, fabsf(x.x)), fabsf(x.y));
            }
            x = sc_cfma(a1, x, s);
        }
        x = sc_cfma(da, xs, x);
        if constexpr (!STATES) {
            // T u
            sc_f16 yt[2] = {zero, zero};
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int k = 0; k < 2 + 2 * q; ++k) {
                    yt[q] = sc_mfma<DT>(tt[2 * q - k + 1], u[k], yt[q]);
                    if constexpr (NP == 2) yt[q] = sc_mfma<DT>(tlo[2 * q - k + 1], u[k], yt[q]);
                }
            // the states as fp16 (re, im) words, scaled by a common power of
            // two, through LDS: lane = mode to lane = block
            const int e = __builtin_amdgcn_readfirstlane(pow2_exp(sc_wave_max(mxv * gf))) - 10;
            float f = ldexpf(gf, -e);
            if (egf - e > 127) {
                // a state so small that f leaves float32 (an input of zeros lets
                // it decay to nothing): scaled value by value
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        sx[t][0][r] = ldexpf(sx[t][0][r] * gf, -e);
                        sx[t][1][r] = ldexpf(sx[t][1][r] * gf, -e);
                    }
                f = 1.f;
            }
#pragma unroll
            for (int n = 0; n < 32; ++n) {
                const int r = 4 * (n >> 3) + (n & 3), t = (n >> 2) & 1;
                xw[SC_PITCH * n + lane] = pack_16x2<F16>(sx[t][0][r] * f, sx[t][1][r] * f);
            }
            settle();
            sc_f16 yx[2] = {zero, zero};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint4 xf = *(const uint4 *)(xw + SC_PITCH * c + 8 * k + 4 * g);
#pragma unroll
                for (int q = 0; q < 2; ++q) yx[q] = sc_mfma<F16>(mxyl[64 * (8 * q + k)], xf, yx[q]);
            }
            settle();
            const float ft = ldexpf(1.f, eT), fx = ldexpf(1.f, e);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float o[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) o[r] = fmaf(yx[q >> 1][8 * (q & 1) + r], fx, yt[q >> 1][8 * (q & 1) + r] * ft);
                *(uint4 *)(frags + 32 * q) = make_uint4(pack_16x2<DT>(o[0], o[1]), pack_16x2<DT>(o[2], o[3]),
                                                        pack_16x2<DT>(o[4], o[5]), pack_16x2<DT>(o[6], o[7]));
            }
            settle();
#pragma unroll
            for (int k = 0; k < 4; ++k)
                store_stream(yp + 512 * k, *(const uint4 *)(lines + 8 * SC_UP * k));
            yp += SC_STEP;
            settle();
        }
    }
    if constexpr (STATES) {
        a.seg[(row * a.nseg + sg) * 64 + lane] = x;
    } else if (a.x_final && s1 == nsteps && on) {
        const long xi = row * a.m + lane;
        const float2 xf = cmul(th, x);
        a.x_final[2 * xi] = xf.x;
        a.x_final[2 * xi + 1] = xf.y;
    }
}

template <int DT, int NP, bool STATES>
hipError_t launch_scan(ScanArgs a, hipStream_t s) {
    const int per_ch = a.B * a.items;
    const int nw = per_ch >= 3 ? 4 : per_ch;
    a.wg_per_ch = (per_ch + nw - 1) / nw;
    const size_t lds = scan_lds<NP, STATES>(nw);
    auto fn = ssm_scan_kernel<DT, NP, STATES>;
    hipLaunchKernelGGL(fn, dim3((unsigned)(a.H * a.wg_per_ch)), dim3(64 * nw), lds, s, a);
    return hipGetLastError();
}

template <int DT, int NP>
hipError_t launch_scan_np(const ScanArgs &a, hipStream_t s) {
    if (a.nseg > 1) {
        ScanArgs b = a;
        b.items = a.nseg - 1;   // the last segment's end state is x_final
        const hipError_t e = launch_scan<DT, NP, true>(b, s);
        if (e != hipSuccess) return e;
    }
    return launch_scan<DT, NP, false>(a, s);
}

}  // namespace

bool ssm_scan_supported(int chunk, int dtype) { return fftconv_mfma_supported(chunk, dtype); }

hipError_t launch_ssm_scan(const void *u, const float *Abar, const float *Bbar, const float *C, const float *D,
                           const float *x0, int B, int H, int L, int m, int dtype, void *y, float *x_final, void *ws,
                           size_t ws_bytes, hipStream_t s) {
    if (L % SC_STEP || m > 64) return hipErrorInvalidValue;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    const long rows = (long)B * H, nsteps = L / SC_STEP;
    // One wave per row while that is one per SIMD or more (B = 1, H = 1024, L =
    // 65536: 97 us, 126 with two segments per row, whose end states take a
    // pass of their own); fewer rows are cut into segments, two waves per SIMD.
    long nseg = 1;
    if (rows < 4L * cus) {
        nseg = (8L * cus + rows - 1) / rows;
        const long room = (long)(ws_bytes / (rows * 64 * sizeof(float2)));
        if (nseg > room) nseg = room;
        if (nseg > nsteps) nseg = nsteps;
        if (nseg < 1) nseg = 1;
    }
    ScanArgs a{};
    a.u = (const uint16_t *)u; a.y = (uint16_t *)y;
    a.Abar = Abar; a.Bbar = Bbar; a.C = C; a.D = D; a.x0 = x0; a.x_final = x_final;
    a.seg = (float2 *)ws;
    a.B = B; a.H = H; a.L = L; a.m = m;
    a.seg_steps = (int)((nsteps + nseg - 1) / nseg);
    a.nseg = (int)((nsteps + a.seg_steps - 1) / a.seg_steps);
    a.items = a.nseg;
    return dtype == BF16 ? launch_scan_np<BF16, 2>(a, s) : launch_scan_np<F16, 1>(a, s);
}

}  // namespace h3
