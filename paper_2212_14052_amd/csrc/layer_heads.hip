// H3 layer with heads of dimension d_h > 1 (Sec. 3.2, Algorithm 1): per head
// h (channels h d_h .. h d_h + d_h - 1) and token t the d_h x d_h outer
// product  KV_t[i][j] = Kbar_t[i] V_t[j]  passes through the diagonal SSM (one
// kernel per entry (h, i, j)), and the head's output is  O_t[j] =
// sum_i Q_t[i] S_t[i][j].  The outer products are d_h^2 sequence rows per head,
// channel (h d_h + i) d_h + j, convolved by the fused FFT convolution like any
// other rows; the two kernels here build them (at the lengths whose convolution
// does not form them in its own loads) and contract them with Q.
#include "common.h"
#include "internal.h"

namespace h3 {
namespace {

__device__ __forceinline__ float ld16(uint16_t v, int dt) { return dt == BF16 ? bf16_to_f32(v) : f16_to_f32(v); }
template <int DT>
__device__ __forceinline__ uint16_t st16(float v) {
    if constexpr (DT == BF16) return __builtin_bit_cast(uint16_t, (__bf16)v);
    else return f32_to_f16(v);
}

// G[b, (h d_h + i) d_h + j, t] = Kbar[b, h d_h + i, t] V[b, h d_h + j, t], one
// rounding; Kbar, V (B, d, L) channel-major, G (B, d d_h, L).  One thread per
// (b, h, 8 consecutive t): d_h + d_h 16-byte loads, d_h^2 16-byte stores.
template <int DT, int DH>
__global__ __launch_bounds__(256) void heads_expand_kernel(const uint16_t *kbar, const uint16_t *v, int B, int d, int L,
                                                           uint16_t *g) {
    const int nh = d / DH, nt = L / 8;
    const long id = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (long)B * nh * nt) return;
    const int t = (int)(id % nt) * 8;
    const long bh = id / nt;
    const int h = (int)(bh % nh), b = (int)(bh / nh);
    float kf[DH][8], vf[DH][8];
#pragma unroll
    for (int i = 0; i < DH; ++i) {
        const long row = ((long)b * d + h * DH + i) * L + t;
        const uint4 kq = *(const uint4 *)(kbar + row), vq = *(const uint4 *)(v + row);
        const uint32_t k4[4] = {kq.x, kq.y, kq.z, kq.w}, v4[4] = {vq.x, vq.y, vq.z, vq.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kf[i][2 * e] = ld16(k4[e] & 0xffffu, DT); kf[i][2 * e + 1] = ld16(k4[e] >> 16, DT);
            vf[i][2 * e] = ld16(v4[e] & 0xffffu, DT); vf[i][2 * e + 1] = ld16(v4[e] >> 16, DT);
        }
    }
#pragma unroll
    for (int i = 0; i < DH; ++i)
#pragma unroll
        for (int j = 0; j < DH; ++j) {
            uint32_t o4[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o4[e] = pack_16x2<DT>(kf[i][2 * e] * vf[j][2 * e], kf[i][2 * e + 1] * vf[j][2 * e + 1]);
            const long row = (((long)b * nh + h) * DH * DH + i * DH + j) * L + t;
            *(uint4 *)(g + row) = make_uint4(o4[0], o4[1], o4[2], o4[3]);
        }
}

// O[b, t, h d_h + j] = sum_i Q[b, h d_h + i, t] S[b, (h d_h + i) d_h + j, t],
// one rounding, written token-major (B, L, d) for the output projection.
// Tile of 64 channels x 64 tokens per 256 threads: thread -> one channel and
// 16 consecutive tokens, then the tile goes through LDS so that the stores are
// 16 bytes along the channels.
template <int DT, int DH>
__global__ __launch_bounds__(256) void heads_contract_kernel(const uint16_t *q, const uint16_t *s, int B, int d, int L,
                                                             uint16_t *o) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[64][64 + 8];   // [token][channel]
    const int ntt = L / 64, nct = d / 64, nh = d / DH;
    const int blk = blockIdx.x;
    const int tt = blk % ntt, ct = (blk / ntt) % nct, b = blk / (ntt * nct);
    const int cl = threadIdx.x >> 2, tq = (threadIdx.x & 3) * 16;
    const int c = ct * 64 + cl, h = c / DH, j = c % DH;
    const int t0 = tt * 64 + tq;
    float acc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int i = 0; i < DH; ++i) {
        const uint16_t *qr = q + ((long)b * d + h * DH + i) * L + t0;
        const uint16_t *sr = s + (((long)b * nh + h) * DH * DH + i * DH + j) * L + t0;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const uint4 qv = *(const uint4 *)(qr + 8 * hh), sv = *(const uint4 *)(sr + 8 * hh);
            const uint32_t q4[4] = {qv.x, qv.y, qv.z, qv.w}, s4[4] = {sv.x, sv.y, sv.z, sv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[8 * hh + 2 * e] += ld16(q4[e] & 0xffffu, DT) * ld16(s4[e] & 0xffffu, DT);
                acc[8 * hh + 2 * e + 1] += ld16(q4[e] >> 16, DT) * ld16(s4[e] >> 16, DT);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) tile[tq + r][cl] = st16<DT>(acc[r]);
    __syncthreads();
    // 64 tokens x 64 channels: thread -> token tk, channels 16 (tid & 3) .. + 15
    const int tk = threadIdx.x >> 2, cq = (threadIdx.x & 3) * 16;
    uint16_t *orow = o + ((long)b * L + tt * 64 + tk) * d + ct * 64 + cq;
    *(uint4 *)orow = *(const uint4 *)&tile[tk][cq];
    *(uint4 *)(orow + 8) = *(const uint4 *)&tile[tk][cq + 8];
}

template <int DT, int DH>
hipError_t launch_heads(const uint16_t *kbar, const uint16_t *v, const uint16_t *q, uint16_t *g, const uint16_t *sv,
                        uint16_t *o, int B, int d, int L, hipStream_t st) {
    if (kbar) {
        const long n = (long)B * (d / DH) * (L / 8);
        hipLaunchKernelGGL((heads_expand_kernel<DT, DH>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, kbar, v, B,
                           d, L, g);
    } else {
        hipLaunchKernelGGL((heads_contract_kernel<DT, DH>), dim3((unsigned)((long)B * (d / 64) * (L / 64))), dim3(256), 0,
                           st, q, sv, B, d, L, o);
    }
    return hipGetLastError();
}

hipError_t launch_heads_any(int dh, const void *kbar, const void *v, const void *q, void *g, const void *sv, void *o,
                            int B, int d, int L, int dtype, hipStream_t s) {
    if (d % 64 || L % 64) return hipErrorInvalidValue;
    const uint16_t *k16 = (const uint16_t *)kbar, *v16 = (const uint16_t *)v, *q16 = (const uint16_t *)q;
    const uint16_t *s16 = (const uint16_t *)sv;
    uint16_t *g16 = (uint16_t *)g, *o16 = (uint16_t *)o;
#define H3_HEADS(DH)                                                                         \
    (dtype == BF16 ? launch_heads<BF16, DH>(k16, v16, q16, g16, s16, o16, B, d, L, s)        \
                   : launch_heads<F16, DH>(k16, v16, q16, g16, s16, o16, B, d, L, s))
    switch (dh) {
        case 2: return H3_HEADS(2);
        case 4: return H3_HEADS(4);
        case 8: return H3_HEADS(8);
    }
#undef H3_HEADS
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_heads_expand(int dh, const void *kbar, const void *v, void *g, int B, int d, int L, int dtype,
                               hipStream_t s) {
    return launch_heads_any(dh, kbar, v, nullptr, g, nullptr, nullptr, B, d, L, dtype, s);
}

hipError_t launch_heads_contract(int dh, const void *q, const void *sv, void *o, int B, int d, int L, int dtype,
                                 hipStream_t s) {
    return launch_heads_any(dh, nullptr, nullptr, q, nullptr, sv, o, B, d, L, dtype, s);
}

}  // namespace h3
