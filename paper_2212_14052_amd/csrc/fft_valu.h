// Float32 FFT engine on the vector ALUs (gfx950): register radix-2/4/8/16
// butterflies, Stockham auto-sorting passes exchanged through LDS.
//
// A length-N signal (N = 2^k, 32 <= N <= 16384) is owned by T = N/16 threads;
// every pass each thread holds 16 complex values (one radix-16 butterfly, or
// 16/R butterflies of a smaller radix R).  Pass (R, Ns) of the Stockham
// decimation-in-time form, butterfly j in [0, N/R):
//     load    v[r] = X[j + r N/R]                          r < R
//     twiddle v[r] *= exp(-2 pi i (j mod Ns) r / (Ns R))
//     DFT_R   on v
//     store   X'[(j div Ns) Ns R + (j mod Ns) + r Ns] = v[r]
// Forward passes: R1 at Ns = 1 (R1 = N / 16^p in {2,4,8}, or 16), then
// radix 16 at Ns = R1, 16 R1, ..., N/16.  The last forward pass leaves
// X[j + r N/16] in thread j's registers, which is exactly what the first pass
// (radix 16, Ns = 1) of a second transform loads, so a pointwise product
// between two transforms needs no LDS exchange.
//
// The DFTs are Cooley-Tukey splits (Sec. 4.1: F_N = P (I (x) F_N1) P^T D
// (I (x) F_N2) P) applied recursively inside the registers; the LDS passes are
// the same factorisation one level up.
#pragma once
#include "common.h"

namespace h3 {

constexpr float kCos16[16] = {
    1.0f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f,
    0.0f, -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f,
    -1.0f, -0.92387953251128674f, -0.70710678118654752f, -0.38268343236508977f,
    0.0f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f};
constexpr float kSin16[16] = {
    0.0f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f,
    1.0f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f,
    0.0f, -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f,
    -1.0f, -0.92387953251128674f, -0.70710678118654752f, -0.38268343236508977f};

// a * exp(-2 pi i j / n) for compile-time-foldable j, n (n divides 16).
__device__ __forceinline__ float2 tw_const(float2 a, int j, int n) {
    int q = (j % n) * (16 / n);
    if (q == 0) return a;
    if (q == 4) return cmul_mi(a);
    if (q == 8) return make_float2(-a.x, -a.y);
    if (q == 12) return cmul_pi(a);
    const float c = kCos16[q], s = -kSin16[q];
    return make_float2(a.x * c - a.y * s, a.x * s + a.y * c);
}

// In-register forward DFT (natural order in and out).
template <int N> struct DFT {
    static __device__ __forceinline__ void run(float2 *v) {
        constexpr int N1 = (N > 4 && N % 4 == 0) ? 4 : 2;
        constexpr int N2 = N / N1;
        float2 A[N1][N2];
#pragma unroll
        for (int n2 = 0; n2 < N2; ++n2) {
            float2 t[N1];
#pragma unroll
            for (int n1 = 0; n1 < N1; ++n1) t[n1] = v[N2 * n1 + n2];
            DFT<N1>::run(t);
#pragma unroll
            for (int k1 = 0; k1 < N1; ++k1) A[k1][n2] = tw_const(t[k1], n2 * k1, N);
        }
#pragma unroll
        for (int k1 = 0; k1 < N1; ++k1) {
            float2 t[N2];
#pragma unroll
            for (int n2 = 0; n2 < N2; ++n2) t[n2] = A[k1][n2];
            DFT<N2>::run(t);
#pragma unroll
            for (int k2 = 0; k2 < N2; ++k2) v[k1 + N1 * k2] = t[k2];
        }
    }
};
template <> struct DFT<1> {
    static __device__ __forceinline__ void run(float2 *) {}
};
template <> struct DFT<2> {
    static __device__ __forceinline__ void run(float2 *v) {
        float2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    }
};
template <> struct DFT<4> {
    static __device__ __forceinline__ void run(float2 *v) {
        float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
        float2 t2 = cadd(v[1], v[3]), t3 = csub(v[1], v[3]);
        v[0] = cadd(t0, t2);
        v[2] = csub(t0, t2);
        v[1] = cadd(t1, cmul_mi(t3));
        v[3] = csub(t1, cmul_mi(t3));
    }
};

constexpr int ilog2c(int n) { return n <= 1 ? 0 : 1 + ilog2c(n / 2); }

__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 4); }

template <int N> struct FFTPlan {
    static constexpr int LOGN = ilog2c(N);
    static constexpr int R1 = (LOGN % 4 == 0) ? 16 : (1 << (LOGN % 4));
    static constexpr int T = N / 16;               // threads per signal
    static constexpr int LDS = N + N / 16;         // float2 per signal (padded)
    static_assert(N >= 32 && N <= 16384, "FFT length out of range");
};

// Pass twiddles exp(-2 pi i jm r / M), jm < Ns = M / R, as constant tables
// evaluated at compile time.  Entry jm holds w1, w2, w3, w4, w8, w12 for
// radix 16 (the other nine are one product of two of them), w1..w4 for radix
// 8, w1 and w2 for radix 4, w1 for radix 2: one to three 16-byte loads per
// butterfly, whole lines across the wave, from a table that stays in the
// vector caches (6 KB for the widest pass at N = 2048).  The transforms are
// bound by VALU issue: w1, w2, w4, w8 from sincospif and up to three products
// each took 3402 VALU instructions for a spectrum and a row pair at N = 2048.
// Entries are the doubles rounded once.
constexpr int kUnit = 16384;   // points on the unit circle
struct UnitOctant {
    double c[kUnit / 8 + 1], s[kUnit / 8 + 1];
};
constexpr UnitOctant make_unit_octant() {   // Taylor series on [0, pi/4]
    UnitOctant t{};
    for (int n = 0; n <= kUnit / 8; ++n) {
        const double x = 6.283185307179586476925286766559 / kUnit * n, x2 = x * x;
        double c = 1.0, s = x, tc = 1.0, ts = x;
        for (int k = 1; k < 10; ++k) {
            tc *= -x2 / ((2.0 * k - 1.0) * (2.0 * k));
            ts *= -x2 / ((2.0 * k) * (2.0 * k + 1.0));
            c += tc;
            s += ts;
        }
        t.c[n] = c;
        t.s[n] = s;
    }
    return t;
}
constexpr UnitOctant kUnitOctant = make_unit_octant();

template <int M, int R> struct PassTab {
    static constexpr int E = R == 16 ? 6 : R == 8 ? 4 : R / 2;   // factors per entry
    alignas(16) float v[M / R * E * 2];
};
template <int M, int R> constexpr PassTab<M, R> make_pass_tab() {
    static_assert(kUnit % M == 0, "pass length out of range");
    PassTab<M, R> t{};
    constexpr int E = PassTab<M, R>::E;
    for (int jm = 0; jm < M / R; ++jm)
        for (int e = 0; e < E; ++e) {
            const int r = R == 16 && e >= 4 ? 4 * (e - 2) : e + 1;   // 1, 2, 3, 4, 8, 12
            const int n = jm * r % M * (kUnit / M), quad = n / (kUnit / 4), m = n % (kUnit / 4);
            const bool sw = m > kUnit / 8;         // past the octant: cos <-> sin
            const int i = sw ? kUnit / 4 - m : m;
            const double c = sw ? kUnitOctant.s[i] : kUnitOctant.c[i];
            const double s = sw ? kUnitOctant.c[i] : kUnitOctant.s[i];
            // exp(-i x) = c - i s, times (-i)^quad
            const double re = quad == 0 ? c : quad == 1 ? -s : quad == 2 ? -c : s;
            const double im = quad == 0 ? -s : quad == 1 ? -c : quad == 2 ? s : c;
            t.v[(jm * E + e) * 2] = (float)re;
            t.v[(jm * E + e) * 2 + 1] = (float)im;
        }
    return t;
}
template <int M, int R> __device__ const PassTab<M, R> kPassTab = make_pass_tab<M, R>();

// The factors of Q butterflies of one pass, loaded ahead of their use.
template <int R> struct PassTw {
    static constexpr int Q = 16 / R, E = PassTab<16 * R, R>::E;
    float2 w[Q * E];
};
template <int N, int R, int Ns>
__device__ __forceinline__ PassTw<R> pass_tw_load(int tid) {
    constexpr int T = N / 16;
    // an opaque index per pass: equal passes of two transforms load their
    // factors again instead of keeping them in registers in between
    asm volatile("" : "+v"(tid));
    PassTw<R> t;
#pragma unroll
    for (int q = 0; q < PassTw<R>::Q; ++q) {
        const int jm = (tid + q * T) & (Ns - 1);
        constexpr int E = PassTw<R>::E;
        if constexpr (E == 1) {
            t.w[q] = ((const float2 *)kPassTab<Ns * R, R>.v)[jm];
        } else {
            const float4 *p = (const float4 *)kPassTab<Ns * R, R>.v + jm * (E / 2);
#pragma unroll
            for (int e = 0; e < E / 2; ++e) {
                const float4 f = p[e];
                t.w[q * E + 2 * e] = make_float2(f.x, f.y);
                t.w[q * E + 2 * e + 1] = make_float2(f.z, f.w);
            }
        }
    }
    return t;
}

// v[r] *= w_r, r = 1..R-1, for one butterfly; e holds its table entry.
template <int R>
__device__ __forceinline__ void pass_twiddles(float2 *v, const float2 *e) {
    float2 w[16];
    w[1] = e[0];
    if (R > 2) w[2] = e[1];
    if (R == 4) w[3] = cmul(w[1], w[2]);
    if (R > 4) {
        w[3] = e[2];
        w[4] = e[3];
    }
    if (R > 8) {
        w[8] = e[4];
        w[12] = e[5];
    }
#pragma unroll
    for (int r = 5; r < R; ++r)
        if (r % 4) w[r] = cmul(w[r % 4], w[r - r % 4]);
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], w[r]);
}

// The largest |row a| and |row b| of a signal of T threads (float bits), from
// each thread's own.  Signals of one wave or less need no LDS; wider ones pass
// one value per wave through red (2 T / 64 words) and one barrier, which also
// ends the reads of LDS before it.
template <int T>
__device__ __forceinline__ void signal_max(uint32_t *red, int tid, uint32_t &a, uint32_t &b) {
    a = group_max<(T < 64 ? T : 64)>(a);
    b = group_max<(T < 64 ? T : 64)>(b);
    if constexpr (T > 64) {
        constexpr int NW = T / 64;
        if ((tid & 63) == 0) {
            red[tid >> 6] = a;
            red[NW + (tid >> 6)] = b;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            a = red[i] > a ? red[i] : a;
            b = red[NW + i] > b ? red[NW + i] : b;
        }
    } else {
        __syncthreads();
    }
}

// Stockham pass pieces for one signal in LDS buffer X (padded indexing).
template <int N, int R>
__device__ __forceinline__ void pass_load(const float2 *X, int tid, float2 *v) {
    constexpr int Q = 16 / R, T = N / 16;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int j = tid + q * T;
#pragma unroll
        for (int r = 0; r < R; ++r) v[q * R + r] = X[lds_pad(j + r * (N / R))];
    }
}

template <int R>
__device__ __forceinline__ void pass_twiddle(const PassTw<R> &t, float2 *v) {
#pragma unroll
    for (int q = 0; q < 16 / R; ++q) pass_twiddles<R>(v + q * R, t.w + q * PassTw<R>::E);
}

template <int R>
__device__ __forceinline__ void pass_dft(float2 *v) {
#pragma unroll
    for (int q = 0; q < 16 / R; ++q) DFT<R>::run(v + q * R);
}

template <int N, int R, int Ns>
__device__ __forceinline__ void pass_store(float2 *X, int tid, const float2 *v) {
    constexpr int Q = 16 / R, T = N / 16;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int j = tid + q * T;
        const int jm = j & (Ns - 1);
        const int base = (j - jm) * R + jm;
#pragma unroll
        for (int r = 0; r < R; ++r) X[lds_pad(base + r * Ns)] = v[q * R + r];
    }
}

// Radix-16 passes with Ns = NS0, 16 NS0, ... while Ns < NSEND (exclusive):
// load, twiddle, DFT, store, barrier.
template <int N, int Ns, int NSEND>
struct MidPasses {
    static __device__ __forceinline__ void run(float2 *X, int tid, float2 *v) {
        if constexpr (Ns < NSEND) {
            const PassTw<16> tw = pass_tw_load<N, 16, Ns>(tid);
            pass_load<N, 16>(X, tid, v);
            pass_twiddle<16>(tw, v);
            pass_dft<16>(v);
            __syncthreads();
            pass_store<N, 16, Ns>(X, tid, v);
            __syncthreads();
            MidPasses<N, Ns * 16, NSEND>::run(X, tid, v);
        }
    }
};

// Forward transform of the signal whose first pass input is already in v
// (thread tid holds X[j + r N/R1] for its butterflies j).  On return thread
// tid holds the spectrum  v[r] = F[tid + r N/16], r < 16.
// Every thread of the workgroup must call this (it contains barriers).
template <int N>
__device__ __forceinline__ void fft_forward_from_regs(float2 *X, int tid, float2 *v) {
    using P = FFTPlan<N>;
    constexpr int R1 = P::R1;
    pass_dft<R1>(v);                         // Ns = 1: no twiddles
    if constexpr (R1 * 16 <= N) {
        pass_store<N, R1, 1>(X, tid, v);
        __syncthreads();
        MidPasses<N, R1, N / 16>::run(X, tid, v);
        // last forward pass: radix 16 at Ns = N/16, result stays in registers
        const PassTw<16> tw = pass_tw_load<N, 16, N / 16>(tid);
        pass_load<N, 16>(X, tid, v);
        pass_twiddle<16>(tw, v);
        pass_dft<16>(v);
    }
}

// Forward transform of a signal whose first pass input is in v laid out as
// the radix-16 pass at Ns = 1 expects (v[r] = X[tid + r N/16]), returning the
// last pass (radix R1 at Ns = N/R1) in registers: thread tid then holds
// F[j + r N/R1] in v[q R1 + r] for its butterflies j = tid + q N/16.
// Used for the second transform of a convolution (the "inverse").
template <int N>
__device__ __forceinline__ void fft_second_from_regs(float2 *X, int tid, float2 *v) {
    using P = FFTPlan<N>;
    constexpr int R1 = P::R1;
    pass_dft<16>(v);                         // radix 16 at Ns = 1
    __syncthreads();                         // LDS may still be read by the previous pass
    pass_store<N, 16, 1>(X, tid, v);
    __syncthreads();
    MidPasses<N, 16, N / R1>::run(X, tid, v);
    const PassTw<R1> tw = pass_tw_load<N, R1, N / R1>(tid);
    pass_load<N, R1>(X, tid, v);
    pass_twiddle<R1>(tw, v);
    pass_dft<R1>(v);
}

}  // namespace h3
