// Kernel and skip gradients of the fused convolution for 16-bit rows, as a
// direct correlation on the matrix cores (L a power of two in 256 .. 8192):
//     dk[h, j] = sum_b sum_{t >= j} dy[b,h,t] u[b,h,t-j],   dD[h] = dk[h, 0].
//
// Why direct: u and dy are 16-bit, so their products are exact in the matrix
// core's float32 and nothing is split, scaled or transformed; L^2/2
// multiply-adds per row cost less there than the transforms do on the VALU.
//
// One tile product.  With rows i < 16, columns n < 16 and a reduction k < 32,
//     D[i][n] += sum_k A[i][k] B[k][n],  A[i][k] = u[x + k - i],
//                                        B[k][n] = dy[x + 256 c + k + 16 n]
// adds to dk[256 c + 16 n + i] the terms t - j = x + k - i.  For a residue
// rho = 32 w the u tiles A_a (x = rho + 256 a) and the dy tiles B_b (at rho +
// 256 b) give every such term as a product of polynomials over 256-blocks:
//     D_c += sum_a A_a B_{a+c},   a + c < NB = L / 256,
// so NB u tiles and NB dy tiles read from LDS feed NB (NB + 1) / 2 matrix
// instructions (528 at L = 8192, against the 1024 of the whole square): the
// kernel is bound by the matrix cores from L = 4096 on, and about equally by
// the LDS reads at 2048.
//
// Split of the work: eight waves per workgroup, one residue each; a workgroup
// walks all rows of its channel and owns the 256-blocks c = kap (mod CS), so
// that few channels still fill the chip and no partial sum reaches memory.
// kap enters as an offset of the dy reads (zeros past the row's end), so
// every kap runs the same code.  The u tiles are held 16 at a time (64
// registers), the dy tiles stream.  A lane's eight u values start at an odd
// element for odd i: five dwords are read and shifted by half a dword.
//
// Accuracy: a float32 accumulator takes at most 64 matrix instructions before
// the eight waves' tiles are added up in LDS and on to a running float32 sum
// (the instruction rounds its accumulator several times: after 256 of them the
// error was 4.7e-7 of the result, after 64 2.3e-7, where the float32
// transforms of the VALU kernel have 2.9e-7).  dD is summed apart, from the
// staged pieces (1e-7).
//
// Measured, dk and dD together (us; the VALU transform kernel before, at 2048
// the fp16 transform kernel with an error of 1e-3): B = 8, H = 768, L = 1024:
// 60 -> 15; L = 2048: 44 -> 31; B = 4, H = 400, L = 4096: 88 -> 35; B = 3, H =
// 400, L = 8192: 321 -> 100.
#include "direct_conv.h"
#include "internal.h"

namespace h3 {
namespace {

typedef _Float16 wg_h8 __attribute__((ext_vector_type(8)));
typedef __bf16 wg_b8 __attribute__((ext_vector_type(8)));
typedef float wg_f4 __attribute__((ext_vector_type(4)));

template <int DT>
__device__ __forceinline__ wg_f4 wg_mfma(uint4 a, uint4 b, wg_f4 c) {
    if constexpr (DT == BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(wg_b8, a), __builtin_bit_cast(wg_b8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(wg_h8, a), __builtin_bit_cast(wg_h8, b), c, 0, 0, 0);
}

// sum of the eight products of two 16-byte pieces, float32
template <int DT>
__device__ __forceinline__ float wg_dot8(uint4 a, uint4 b) {
    const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (DT == BF16) {
            s = fmaf(__uint_as_float(x[i] << 16), __uint_as_float(y[i] << 16), s);
            s = fmaf(__uint_as_float(x[i] & 0xffff0000u), __uint_as_float(y[i] & 0xffff0000u), s);
        } else {
            s = fmaf(f16_to_f32((uint16_t)x[i]), f16_to_f32((uint16_t)y[i]), s);
            s = fmaf(f16_to_f32((uint16_t)(x[i] >> 16)), f16_to_f32((uint16_t)(y[i] >> 16)), s);
        }
    }
    return s;
}

constexpr int WG_NT = 512, WG_NW = 8;

// Shapes of one instance: rows staged at once, LDS elements per u and dy row
// (16 zeros before u; zeros past dy for the columns and kap), bytes per stage.
template <int NB, int CS>
struct WgPlan {
    static constexpr int L = 256 * NB;
    static constexpr int R = L >= 4096 ? 1 : (4096 / L < 4 ? 4096 / L : 4);
    static constexpr int US = L + 24, DS = L + 256 * CS;
    static constexpr int STAGE = R * (US + DS) * 2;
    static constexpr int NT = NB / CS;                  // accumulator tiles
    static constexpr int TR = NT < 4 ? NT : 4;          // tiles per reduction round
    static constexpr int AB = NB < 16 ? NB : 16;        // u tiles held at once
    static constexpr int FLUSH = 64 / NB;               // rows between reductions
    static constexpr size_t LDS = 2 * (size_t)STAGE + (size_t)WG_NW * TR * 1024;
    // waves per SIMD the registers are allotted for
    static constexpr int WPE = NB <= 8 ? 4 : 2;
};

template <int DT, int NB, int CS>
__global__ __launch_bounds__(WG_NT, (WgPlan<NB, CS>::WPE)) void wgrad_direct_kernel(const uint16_t *u, const uint16_t *dy,
                                                                                 int B, int H, float *dk, float *dD) {
    using P = WgPlan<NB, CS>;
    constexpr int L = P::L, R = P::R, NT = P::NT, TR = P::TR;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float *red = (float *)(smem + 2 * P::STAGE);   // [wave][TR * 256]
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int blk = xcd_logical_block(blockIdx.x, gridDim.x);
    const int h = blk / CS, kap = blk % CS;
    const int i16 = lane & 15, g = lane >> 4;

    auto urow = [&](int buf, int r) { return (uint16_t *)(smem + buf * P::STAGE) + r * (P::US + P::DS); };
    auto drow = [&](int buf, int r) { return urow(buf, r) + P::US; };

    // the zeros around the rows (staging never writes them)
    for (int br = 0; br < 2 * R; ++br) {
        uint16_t *ur = urow(br / R, br % R), *dr = drow(br / R, br % R);
        for (int x = tid; x < 24; x += WG_NT) ur[x < 16 ? x : L + x] = 0;
        for (int x = tid; x < 256 * CS; x += WG_NT) dr[L + x] = 0;
    }

    // staging: 16-byte pieces of R u rows and R dy rows, one stage ahead
    constexpr int PIECES = R * L / 8;                       // per operand
    constexpr int PT = (PIECES + WG_NT - 1) / WG_NT;
    uint4 su[PT], sd[PT];
    auto fetch = [&](int b0) {
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int q = p * WG_NT + tid, r = q / (L / 8), x = q % (L / 8);
            if (q < PIECES && b0 + r < B) {
                const long o = ((long)(b0 + r) * H + h) * L + 8 * x;
                su[p] = *(const uint4 *)(u + o);
                sd[p] = *(const uint4 *)(dy + o);
            }
        }
    };
    auto stash = [&](int buf, int b0) {
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int q = p * WG_NT + tid, r = q / (L / 8), x = q % (L / 8);
            if (q < PIECES && b0 + r < B) {
                *(uint4 *)(urow(buf, r) + 16 + 8 * x) = su[p];
                *(uint4 *)(drow(buf, r) + 8 * x) = sd[p];
            }
        }
    };

    wg_f4 acc[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) acc[c] = wg_f4{0.f, 0.f, 0.f, 0.f};
    // the lane's element offsets: u (16 zeros in front) and dy
    const int e0 = 16 + 32 * w + 8 * g - i16;
    const int ud = e0 >> 1;
    const uint32_t sh = (uint32_t)(e0 & 1) * 16;
    const int d0 = 256 * kap + 32 * w + 16 * i16 + 8 * g;

    constexpr int OPT = TR >= 2 ? TR / 2 : 1;   // outputs per thread and round
    constexpr int ROUNDS = NT / TR;
    float own[ROUNDS][OPT];
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q)
#pragma unroll
        for (int o = 0; o < OPT; ++o) own[q][o] = 0.f;

    // dD: the products of the staged pieces, in float32
    float dd = 0.f;
    auto dot = [&](int b0) {
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            const int q = p * WG_NT + tid, r = q / (L / 8);
            if (q < PIECES && b0 + r < B) dd += wg_dot8<DT>(su[p], sd[p]);
        }
    };

    fetch(0);
    stash(0, 0);
    if (kap == 0) dot(0);
    __syncthreads();
    int since = 0;
    for (int b0 = 0, buf = 0; b0 < B; b0 += R, buf ^= 1) {
        const bool more = b0 + R < B;
        if (more) fetch(b0 + R);
        const int nr = min(R, B - b0);
        for (int r = 0; r < nr; ++r) {
            const uint32_t *up = (const uint32_t *)urow(buf, r) + ud;
            const uint16_t *dp = drow(buf, r) + d0;
#pragma unroll
            for (int a0 = 0; a0 < NB; a0 += P::AB) {
                uint4 A[P::AB];
#pragma unroll
                for (int a = 0; a < P::AB; ++a) A[a] = cd_frag(up + 128 * (a0 + a), sh);
#pragma unroll
                for (int b = a0; b < NB; ++b) {
                    const uint4 Bv = *(const uint4 *)(dp + 256 * b);
#pragma unroll
                    for (int a = 0; a < P::AB; ++a)
                        if (a0 + a <= b && (b - a0 - a) % CS == 0)
                            acc[(b - a0 - a) / CS] = wg_mfma<DT>(A[a], Bv, acc[(b - a0 - a) / CS]);
                }
            }
        }
        since += R;
        if (!more || since + R > P::FLUSH) {
            since = 0;
            // add the eight waves' tiles, TR at a time, on to the running sums
#pragma unroll
            for (int q = 0; q < ROUNDS; ++q) {
                // lane: rows 4 g .. + 3 of column i16 -> dk offsets 16 i16 + 4 g .. + 3
#pragma unroll
                for (int c = 0; c < TR; ++c) {
                    *(wg_f4 *)(red + (w * TR + c) * 256 + 16 * i16 + 4 * g) = acc[q * TR + c];
                    acc[q * TR + c] = wg_f4{0.f, 0.f, 0.f, 0.f};
                }
                __syncthreads();
                if (tid * OPT < TR * 256) {
#pragma unroll
                    for (int o = 0; o < OPT; ++o) {
                        float s = 0.f;
#pragma unroll
                        for (int v = 0; v < WG_NW; ++v) s += red[v * TR * 256 + tid * OPT + o];
                        own[q][o] += s;
                    }
                }
                __syncthreads();
            }
        }
        if (more) {
            stash(buf ^ 1, b0 + R);
            if (kap == 0) dot(b0 + R);
            __syncthreads();
        }
    }
    if (tid * OPT < TR * 256) {
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const int o = tid * OPT;
            const int j = 256 * (CS * (q * TR + o / 256) + kap) + o % 256;
            if (dk) {
#pragma unroll
                for (int e = 0; e < OPT; ++e) dk[(long)h * L + j + e] = own[q][e];
            }
        }
    }
    if (dD && kap == 0) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) dd += __shfl_xor(dd, o, 64);
        if (lane == 0) red[w] = dd;   // the last reduction's reads are done
        __syncthreads();
        if (tid == 0) {
            float s = 0.f;
            for (int v = 0; v < WG_NW; ++v) s += red[v];
            dD[h] = s;
        }
    }
}

template <int DT, int NB, int CS>
hipError_t launch_direct(const uint16_t *u, const uint16_t *dy, int B, int H, float *dk, float *dD, hipStream_t s) {
    using P = WgPlan<NB, CS>;
    auto fn = wgrad_direct_kernel<DT, NB, CS>;
    if (P::LDS > 65536)
        (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)P::LDS);
    hipLaunchKernelGGL(fn, dim3((unsigned)H * CS), dim3(WG_NT), P::LDS, s, u, dy, B, H, dk, dD);
    return hipGetLastError();
}

template <int DT, int NB>
hipError_t launch_direct_cs(const uint16_t *u, const uint16_t *dy, int B, int H, float *dk, float *dD, hipStream_t s) {
    // Few channels: more workgroups per channel, each with fewer 256-blocks
    // (measured in us with CS = 1 / 2 / 4: L = 4096, B = 16, H = 64: 56 / 38 /
    // 30; B = 4, H = 400: 35 / 35 / 46.  L = 8192, B = 16, H = 64: 266 / 112 /
    // 82; B = 3, H = 400: 139 / 100 / 115, where CS = 1 spills registers).
    if constexpr (NB >= 16) {
        if (H <= (NB == 32 ? 128 : 64)) return launch_direct<DT, NB, 4>(u, dy, B, H, dk, dD, s);
    }
    if constexpr (NB == 32) return launch_direct<DT, NB, 2>(u, dy, B, H, dk, dD, s);
    if constexpr (NB == 16) {
        if (H <= 128) return launch_direct<DT, NB, 2>(u, dy, B, H, dk, dD, s);
    }
    if constexpr (NB < 32) return launch_direct<DT, NB, 1>(u, dy, B, H, dk, dD, s);
}

template <int DT>
hipError_t launch_direct_dt(const uint16_t *u, const uint16_t *dy, int B, int H, int L, float *dk, float *dD,
                            hipStream_t s) {
    switch (L) {
        case 256: return launch_direct_cs<DT, 1>(u, dy, B, H, dk, dD, s);
        case 512: return launch_direct_cs<DT, 2>(u, dy, B, H, dk, dD, s);
        case 1024: return launch_direct_cs<DT, 4>(u, dy, B, H, dk, dD, s);
        case 2048: return launch_direct_cs<DT, 8>(u, dy, B, H, dk, dD, s);
        case 4096: return launch_direct_cs<DT, 16>(u, dy, B, H, dk, dD, s);
        case 8192: return launch_direct_cs<DT, 32>(u, dy, B, H, dk, dD, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool wgrad_direct_supported(int L, int dtype) {
    return (dtype == F16 || dtype == BF16) && L >= 256 && L <= 8192 && (L & (L - 1)) == 0;
}

hipError_t launch_wgrad_direct(const void *u, const void *dy, int B, int H, int L, int dtype, float *dk, float *dD,
                               hipStream_t s) {
    const uint16_t *u16 = (const uint16_t *)u, *d16 = (const uint16_t *)dy;
    return dtype == BF16 ? launch_direct_dt<BF16>(u16, d16, B, H, L, dk, dD, s)
                         : launch_direct_dt<F16>(u16, d16, B, H, L, dk, dD, s);
}

}  // namespace h3
