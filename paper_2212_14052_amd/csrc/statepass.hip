// State passing (Sec. 4.2, Algorithm 2) pieces, gfx950.
//
// With chunk length N' and the state x^(c) carried into chunk c (the state
// after the previous chunk's last input):
//   end-of-chunk contribution  s_c = M_ux u^(c),  M_ux[n, i] = Abar_n^{N'-1-i} Bbar_n
//   state update               x^(c+1) = Abar^{N'} x^(c) + s_c
//   output                     y^(c)_t = (f * u^(c))_t + D u^(c)_t
//                                        + 2 Re sum_n C_n Abar_n^{t+1} x^(c)_n
// The chunk-local sums s_c of all chunks are independent (one workgroup per
// chunk row); only the short scan over chunks is sequential.  16-bit I/O at
// chunks 2048, 8192 and 16384 takes the one-pass kernel of ssm_scan.hip
// instead; this file serves float32 I/O and the other chunks.
#include "common.h"
#include "internal.h"

namespace h3 {

// ----------------------------------------------------------- chunk sums ----
// s_c[n] = Bbar_n sum_i Abar_n^{N'-1-i} u_i, factorised with i = T a + b:
//   s_c[n] = Bbar_n sum_a Abar_n^{N' - T(a+1)} R[a][n],
//   R[a][n] = sum_{b<T} Abar_n^{T-1-b} u_{T a + b}.
constexpr int CS_T = 64;
constexpr int CS_THREADS = 256;

template <int DT>
__global__ __launch_bounds__(CS_THREADS) void chunk_states_kernel(const void *u_, const float *Abar,
                                                                  const float *Bbar, int H, int L,
                                                                  int m, int chunk, float2 *states) {
    using io = IO<DT>;
    typedef typename io::T T_;
    const T_ *u = (const T_ *)u_;
    extern __shared__ float smem[];
    float *us = smem;                                   // chunk of u, float32
    float2 *Qs = (float2 *)(smem + chunk);              // [b][n] Abar_n^{T-1-b}
    float2 *red = Qs + CS_T * H3_MAX_MODES_DEV;         // [4][n] partial sums
    const int nchunk = L / chunk;
    const int crow = blockIdx.x;                        // (b*H + h) * nchunk + c
    const int row = crow / nchunk, c = crow % nchunk;
    const int h = row % H;
    const int tid = threadIdx.x;
    const long base = (long)row * L + (long)c * chunk;
    for (int i = tid; i < chunk; i += CS_THREADS) us[i] = io::ld(u, base + i);
    const int T = chunk < CS_T ? chunk : CS_T;
    const int NA = chunk / T;
    const int n = tid % H3_MAX_MODES_DEV, g = tid / H3_MAX_MODES_DEV;
    double lr = 0, li = 0;
    if (n < m) {
        const long i = (long)h * m + n;
        const double ar = Abar[2 * i], ai = Abar[2 * i + 1];
        lr = 0.5 * log(ar * ar + ai * ai);
        li = atan2(ai, ar);
        for (int b = g; b < T; b += CS_THREADS / H3_MAX_MODES_DEV)
            Qs[b * H3_MAX_MODES_DEV + n] = cexp_scaled((double)(T - 1 - b), lr, li);
    }
    __syncthreads();
    float2 acc = make_float2(0.f, 0.f);
    if (n < m) {
        constexpr int G = CS_THREADS / H3_MAX_MODES_DEV;     // 4 groups over a
        // a = g + G i, i descending, so the anchor power grows in magnitude:
        // exponent N' - T(a+1) increases by G T per step.
        int alast = g + G * ((NA - 1 - g) / G);
        if (g < NA) {
            float2 pw = cexp_scaled((double)(chunk - T * (alast + 1)), lr, li);
            const float2 step = cexp_scaled((double)(G * T), lr, li);
            for (int a = alast; a >= 0; a -= G) {
                float rr = 0.f, ri = 0.f;
                const float *ua = us + T * a;
                for (int b = 0; b < T; ++b) {
                    const float2 q = Qs[b * H3_MAX_MODES_DEV + n];
                    const float x = ua[b];
                    rr = fmaf(q.x, x, rr);
                    ri = fmaf(q.y, x, ri);
                }
                acc = cadd(acc, cmul(pw, make_float2(rr, ri)));
                pw = cmul(pw, step);
            }
        }
    }
    red[g * H3_MAX_MODES_DEV + n] = acc;
    __syncthreads();
    if (g == 0 && n < m) {
        float2 s = red[n];
        for (int k = 1; k < CS_THREADS / H3_MAX_MODES_DEV; ++k) s = cadd(s, red[k * H3_MAX_MODES_DEV + n]);
        const long i = (long)h * m + n;
        const float2 bb = make_float2(Bbar[2 * i], Bbar[2 * i + 1]);
        states[(long)crow * m + n] = cmul(bb, s);
    }
}

// ------------------------------------------------- chunk sums, MFMA form ---
// Same sums for 16-bit input and chunk 1024 or 4096.  Per channel, with blocks
// of BW = 128 inputs (64 at chunk 1024),
//   R[n][a] = sum_{b<BW} Abar_n^{BW-1-b} u_{BW a + b}
// is a real matrix product (rows: Re / Im of 64 modes; reduction b; columns
// a = 0 .. N'/BW - 1) on 16x16x32 MFMAs with the powers in 16-bit and the
// input as it is stored; then
//   s[n] = Bbar_n sum_a Abar_n^{N' - BW (a + 1)} R[n][a]
// in fp32 with the weights held in registers (powers in float64 first).  The
// second sum is the VALU's share (a complex multiply-add and a weight update
// per mode and column), so the wider block halves it at the same matrix-core
// work.
// Workgroup: one channel and a set of its chunk rows; wave w owns modes
// 16 w .. 16 w + 15 (row tile w of the real parts, w + 4 of the imaginary).
// Chunk rows reach LDS without passing through registers: the four waves copy
// 1 KB slices of a row (64 lanes x 16 bytes, lane i to byte 16 i of the
// slice) with global_load_lds_dwordx4 into two row buffers, one row ahead of
// the row being reduced.  A row is staged as N'/BW LDS rows of
// BW inputs (2 BW bytes, 16-byte chunks), chunk c of LDS row a at slot
// c ^ ((a / (256 / 2 BW)) % (2 BW / 16)), so the 16 lanes of an operand read
// (16 consecutive rows a, one chunk) hit 16 distinct 16-byte bank groups.
// Each row's 64 end-state sums go to LDS; wave 0 stores them after the next
// barrier.
typedef _Float16 sp_h8 __attribute__((ext_vector_type(8)));
typedef __bf16 sp_b8 __attribute__((ext_vector_type(8)));
typedef float sp_f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 sp_zmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 sp_zpow(double2 z, int e) {
    double2 r = make_double2(1.0, 0.0);
    while (e) {
        if (e & 1) r = sp_zmul(r, z);
        z = sp_zmul(z, z);
        e >>= 1;
    }
    return r;
}

template <int DT>
__device__ __forceinline__ sp_f4 sp_mfma(uint4 a, uint4 b, sp_f4 c) {
    if constexpr (DT == BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(sp_b8, a), __builtin_bit_cast(sp_b8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(sp_h8, a), __builtin_bit_cast(sp_h8, b), c, 0, 0, 0);
}
// (the empty asm keeps a float that came from a double opaque: otherwise the
// two roundings fold into one float64 -> 16-bit conversion, a long integer
// sequence instead of one instruction)
template <int DT>
__device__ __forceinline__ uint32_t sp_pack(float lo, float hi) {
    asm("" : "+v"(lo), "+v"(hi));
    if constexpr (DT == BF16) {
        typedef __bf16 b2 __attribute__((ext_vector_type(2)));
        b2 v = {(__bf16)lo, (__bf16)hi};
        return __builtin_bit_cast(uint32_t, v);
    } else {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        h2 v = {(_Float16)lo, (_Float16)hi};
        return __builtin_bit_cast(uint32_t, v);
    }
}

constexpr int CS_NS = 2;   // row buffers in the copy ring

typedef __attribute__((address_space(3))) void cs_lds_t;

// LDS bytes for a chunk: the row ring, the results [2][64] float2 and a 1 KB
// slot for the copies of waves with one slice less
size_t chunk_states_lds(int chunk) { return (size_t)CS_NS * chunk * 2 + 2 * 64 * 8 + 1024; }

template <int DT, int BW, int CHUNK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void chunk_states_mfma(
    const uint16_t *u, const float *Abar, const float *Bbar, int B, int H, int L, int m, int wg_per_ch,
    float2 *states) {
    constexpr int chunk = CHUNK;
    constexpr int KS = BW / 32;          // 32-wide reduction steps per block
    constexpr int RB = 2 * BW;           // bytes per LDS row
    constexpr int SPR = RB / 16;         // 16-byte slots per LDS row
    constexpr int RPB = 256 / RB;        // LDS rows per 256-byte bank row
    extern __shared__ __attribute__((aligned(1024))) char cs_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // the wave index, in a scalar register
    const int r16 = lane & 15, kg = lane >> 4;
    const int h = blockIdx.x / wg_per_ch, part = blockIdx.x % wg_per_ch;
    const int nchunk = L / chunk;
    constexpr int NCT = chunk / BW / 16;   // column tiles
    static_assert(chunk / BW % 16 == 0, "whole column tiles");
    const int rows_per_ch = B * nchunk;
    const int per = (rows_per_ch + wg_per_ch - 1) / wg_per_ch;
    const int r0 = part * per, r1 = min(r0 + per, rows_per_ch);
    if (r0 >= r1) return;   // uniform over the workgroup
    const int row_b = chunk * 2;                 // bytes of a staged row
    float2 *res = (float2 *)(cs_lds + CS_NS * row_b);   // [2][64]
    const uint32_t lds0 = (uint32_t)(uintptr_t)(cs_lds_t *)cs_lds;
    const uint32_t dummy = lds0 + (uint32_t)(CS_NS * row_b + 2 * 64 * 8);

    // A operand (powers, 16-bit): rows n = 16 w + r16, reduction b = 32 ks + 8 kg + i
    uint4 Are[KS], Aim[KS];
    {
        const int n = 16 * w + r16;
        double2 z = make_double2(0.0, 0.0);
        if (n < m) z = make_double2(Abar[2 * ((long)h * m + n)], Abar[2 * ((long)h * m + n) + 1]);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            // b from 32 ks + 8 kg + 7 down to 32 ks + 8 kg: exponents BW - 1 - b ascending
            double2 p = sp_zpow(z, BW - 1 - (32 * ks + 8 * kg + 7));
            float pr[8], pi[8];
#pragma unroll
            for (int i = 7; i >= 0; --i) {
                pr[i] = (float)p.x;
                pi[i] = (float)p.y;
                p = sp_zmul(p, z);
            }
            Are[ks] = make_uint4(sp_pack<DT>(pr[0], pr[1]), sp_pack<DT>(pr[2], pr[3]), sp_pack<DT>(pr[4], pr[5]), sp_pack<DT>(pr[6], pr[7]));
            Aim[ks] = make_uint4(sp_pack<DT>(pi[0], pi[1]), sp_pack<DT>(pi[2], pi[3]), sp_pack<DT>(pi[4], pi[5]), sp_pack<DT>(pi[6], pi[7]));
        }
    }
    // E weights for the lane's outputs: modes n = 16 w + 4 kg + j, columns
    // a = 16 ct + r16, weight Abar_n^{chunk - BW (a + 1)}.  Column tiles run
    // from the last down, the weight growing by Abar_n^{16 BW} per tile (fp32;
    // the starting weight and the step in float64 first).
    float2 E0[4], Zstep[4];
    float2 Bb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = 16 * w + 4 * kg + j;
        double2 z = make_double2(0.0, 0.0);
        Bb[j] = make_float2(0.f, 0.f);
        if (n < m) {
            const long i = (long)h * m + n;
            z = make_double2(Abar[2 * i], Abar[2 * i + 1]);
            Bb[j] = make_float2(Bbar[2 * i], Bbar[2 * i + 1]);
        }
        const double2 zstep = sp_zpow(z, 16 * BW);
        const double2 p = sp_zpow(z, chunk - BW * (16 * (NCT - 1) + r16 + 1));
        E0[j] = make_float2((float)p.x, (float)p.y);
        Zstep[j] = make_float2((float)zstep.x, (float)zstep.y);
    }

    // this wave's slices q = w + 4 s of a staged row (s < nsl; waves past the
    // last slice copy slice w again into the never-read slot): the lane's
    // source element within the chunk row
    const int slices = row_b / 1024;             // chunk % 512 == 0
    const int nsl = (slices + 3) / 4;            // copies per wave per row (1..8)
    auto src_elem = [&](int q) {
        const int b = 1024 * q + 16 * lane;
        const int a = b / RB, slot = (b % RB) / 16;
        const int c = slot ^ ((a / RPB) % SPR);
        return BW * a + 8 * c;
    };
    // copies of chunk row rr into buffer (rr - r0) % CS_NS
    auto issue = [&](int rr) {
        const int bb = rr / nchunk, cc = rr % nchunk;
        // the row's address and the buffer, in scalar registers (wave-uniform)
        const uint64_t sp = (uint64_t)(uintptr_t)(u + ((long)bb * H + h) * L + (long)cc * chunk);
        const uint64_t spu = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(sp >> 32)) << 32) |
                             (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)sp);
        const uint16_t *src = (const uint16_t *)(uintptr_t)spu;
        const uint32_t st = lds0 + (uint32_t)(((rr - r0) % CS_NS) * row_b);
        for (int sl = 0; sl < nsl; ++sl) {
            const int q = w + 4 * sl;
            const bool real = q < slices;
            const uint32_t vo = 2u * (uint32_t)src_elem(real ? q : w);
            const uint32_t la = __builtin_amdgcn_readfirstlane(real ? st + (uint32_t)q * 1024 : dummy);
            asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, %2"
                         :
                         : "v"(vo), "s"(la), "s"(src)
                         : "memory", "m0");
        }
    };
    auto store_row = [&](int rr) {   // wave 0: the 64 sums of row rr from res[(rr - r0) & 1]
        const int bb = rr / nchunk, cc = rr % nchunk;
        const long crow = ((long)bb * H + h) * nchunk + cc;
        if (lane < m) states[crow * m + lane] = res[((rr - r0) & 1) * 64 + lane];
    };

    issue(r0);
    for (int rr = r0; rr < r1; ++rr) {
        // this row's copies landed for this wave, then for every wave; the
        // reads of the buffer refilled below (the previous row's) are done.
        // lgkmcnt(0) as well: the previous row's sums, written to res by
        // every wave, must have reached LDS before wave 0 reads them below
        // (a barrier alone does not wait for LDS writes in flight)
        __builtin_amdgcn_s_waitcnt(0x070);   // vmcnt(0) lgkmcnt(0)
        asm volatile("s_barrier" ::: "memory");
        if (w == 0 && rr > r0) store_row(rr - 1);
        // the next row's copies
        if (rr + 1 < r1) issue(rr + 1);
        const char *us = cs_lds + ((rr - r0) % CS_NS) * row_b;
        sp_f4 sre = {0.f, 0.f, 0.f, 0.f}, sim = {0.f, 0.f, 0.f, 0.f};
        float2 E[4] = {E0[0], E0[1], E0[2], E0[3]};
#pragma unroll
        for (int ct = NCT - 1; ct >= 0; --ct) {
            sp_f4 accr = {0.f, 0.f, 0.f, 0.f}, acci = {0.f, 0.f, 0.f, 0.f};
            const int a = 16 * ct + r16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                // B operand: column a, reduction b = 32 ks + 8 kg .. + 7 (16-byte chunk 4 ks + kg)
                const int c = 4 * ks + kg;
                const uint4 bv = *(const uint4 *)(us + a * RB + 16 * (c ^ ((a / RPB) % SPR)));
                accr = sp_mfma<DT>(Are[ks], bv, accr);
                acci = sp_mfma<DT>(Aim[ks], bv, acci);
            }
            // lane: rows (modes) 4 kg + j, column a = 16 ct + r16
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sre[j] = fmaf(E[j].x, accr[j], fmaf(-E[j].y, acci[j], sre[j]));
                sim[j] = fmaf(E[j].x, acci[j], fmaf(E[j].y, accr[j], sim[j]));
                E[j] = cmul(E[j], Zstep[j]);
            }
        }
        // reduce over the 16 columns held by lanes r16 = 0..15
#pragma unroll
        for (int o = 1; o < 16; o <<= 1)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sre[j] += __shfl_xor(sre[j], o);
                sim[j] += __shfl_xor(sim[j], o);
            }
        if (r16 == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                res[((rr - r0) & 1) * 64 + 16 * w + 4 * kg + j] = cmul(Bb[j], make_float2(sre[j], sim[j]));
        }
    }
    __syncthreads();   // the last row's sums are in LDS; every copy has landed
    if (w == 0) store_row(r1 - 1);
}

bool chunk_states_mfma_ok(int chunk, int dtype) {
    return (dtype == F16 || dtype == BF16) && (chunk == 1024 || chunk == 4096);
}

hipError_t launch_chunk_states_mfma(const void *u, const float *Abar, const float *Bbar, int B, int H,
                                    int L, int m, int chunk, int dtype, float2 *states, hipStream_t s) {
    const int rows_per_ch = B * (L / chunk);
    const uint16_t *u16 = (const uint16_t *)u;
    const size_t lds = chunk_states_lds(chunk);
    // Workgroups per channel: a workgroup walks its rows one after another,
    // the grid runs in ceil(workgroups / resident) rounds.  Take the count in
    // 1..8 (at least 4 rows each where the channel has them) that minimises
    // rounds x (rows per workgroup + 1), the 1 standing for a workgroup's
    // set-up (its power tables in float64).
    auto pick_wg = [&](const void *fn) {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 256, lds) != hipSuccess || per_cu < 1) per_cu = 1;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 1;
        const long resident = (long)per_cu * cus;
        int best = 1;
        long best_cost = -1;
        for (int w = 1; w <= 8; ++w) {
            if (w > 1 && rows_per_ch < 4 * w) break;
            const long rounds = ((long)H * w + resident - 1) / resident;
            const long cost = rounds * ((rows_per_ch + w - 1) / w + 1);
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = w;
            }
        }
        return best;
    };
#define H3_CS_LAUNCH(DTV, BWV, CV)                                                                               \
    do {                                                                                                         \
        auto fn = chunk_states_mfma<DTV, BWV, CV>;                                                               \
        (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);      \
        const int wg = pick_wg((const void *)fn);                                                                \
        hipLaunchKernelGGL(fn, dim3(H * wg), dim3(256), lds, s, u16, Abar, Bbar, B, H, L, m, wg, states);        \
    } while (0)
    if (dtype == BF16) {
        if (chunk == 4096) H3_CS_LAUNCH(BF16, 128, 4096);
        else H3_CS_LAUNCH(BF16, 64, 1024);
    } else {
        if (chunk == 4096) H3_CS_LAUNCH(F16, 128, 4096);
        else H3_CS_LAUNCH(F16, 64, 1024);
    }
#undef H3_CS_LAUNCH
    return hipGetLastError();
}

// ------------------------------------------------------------------ scan ---
// One thread per (row, mode): x <- Abar^{N'} x + s_c across the chunks.
// Writes corr_W[row, c, n] = C_n x^(c)_n Abar_n (so that the initial-state
// term of chunk c is 2 Re sum_n corr_W Abar_n^t) and x_final = x^(nchunk).
__global__ void state_scan_kernel(const float *Abar, const float *C, const float *x0,
                                  const float2 *states, int B, int H, int m, int chunk, int nchunk,
                                  float2 *corr_W, float *x_final) {
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= (long)B * H * m) return;
    const int n = (int)(gid % m);
    const long row = gid / m;
    const int h = (int)(row % H);
    const long i = (long)h * m + n;
    const double ar = Abar[2 * i], ai = Abar[2 * i + 1];
    const float2 ab = make_float2((float)ar, (float)ai);
    const float2 cc = make_float2(C[2 * i], C[2 * i + 1]);
    const float2 cab = cmul(cc, ab);
    const float2 AN = cexp_scaled((double)chunk, 0.5 * log(ar * ar + ai * ai), atan2(ai, ar));
    float2 x = x0 ? make_float2(x0[2 * gid], x0[2 * gid + 1]) : make_float2(0.f, 0.f);
    for (int c = 0; c < nchunk; ++c) {
        const long ci = (row * nchunk + c) * m + n;
        corr_W[ci] = cmul(cab, x);
        x = cadd(cmul(AN, x), states[ci]);
    }
    if (x_final) {
        x_final[2 * gid] = x.x;
        x_final[2 * gid + 1] = x.y;
    }
}

hipError_t launch_chunk_states(const void *u, const float *Abar, const float *Bbar, int B, int H,
                               int L, int m, int chunk, int dtype, float2 *states, hipStream_t s) {
    if (chunk_states_mfma_ok(chunk, dtype))
        return launch_chunk_states_mfma(u, Abar, Bbar, B, H, L, m, chunk, dtype, states, s);
    const int nchunk = L / chunk;
    const long ncr = (long)B * H * nchunk;
    const size_t lds = (size_t)chunk * sizeof(float) +
                       (size_t)(CS_T + CS_THREADS / H3_MAX_MODES_DEV) * H3_MAX_MODES_DEV * sizeof(float2);
    dim3 grid((unsigned)ncr), block(CS_THREADS);
    if (lds > 65536) {
        (void)hipFuncSetAttribute((const void *)chunk_states_kernel<F32>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        (void)hipFuncSetAttribute((const void *)chunk_states_kernel<F16>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        (void)hipFuncSetAttribute((const void *)chunk_states_kernel<BF16>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    }
    switch (dtype) {
        case F32:
            hipLaunchKernelGGL(chunk_states_kernel<F32>, grid, block, lds, s, u, Abar, Bbar, H, L, m, chunk, states);
            break;
        case F16:
            hipLaunchKernelGGL(chunk_states_kernel<F16>, grid, block, lds, s, u, Abar, Bbar, H, L, m, chunk, states);
            break;
        case BF16:
            hipLaunchKernelGGL(chunk_states_kernel<BF16>, grid, block, lds, s, u, Abar, Bbar, H, L, m, chunk, states);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_state_scan(const float *Abar, const float *C, const float *x0,
                             const float2 *states, int B, int H, int m, int chunk, int nchunk,
                             float2 *corr_W, float *x_final, hipStream_t s) {
    const long n = (long)B * H * m;
    hipLaunchKernelGGL(state_scan_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Abar, C,
                       x0, states, B, H, m, chunk, nchunk, corr_W, x_final);
    return hipGetLastError();
}

}  // namespace h3
