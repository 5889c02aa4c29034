// a5/a6 on the matrix cores: fused fiber gather + prediction + residual +
// gradient contraction, FP32 in and out, v_mfma_f32_16x16x4_f32.
//
// Two forms, both with blocks of four wavefronts on 64 rows of G_{n(2)} (16
// per wavefront) and a group of samples, the g tile in accumulators over the
// group and written once as a partial sum; partials are added in a fixed
// order afterwards.
//
// Streaming form (any R_n R_{n+1}, any number of samples per group), chunks
// of 64 samples:
//   GEMM1  P^T = S G^T    (64 x 16, K = R_n R_{n+1})  A = S (LDS), B = the
//                                                     wavefront's rows of G
//                                                     (registers, loaded once)
//   E      = X_F - P      scaled by -1/(m J_n p_f)
//   GEMM2  g += E S       (16 x RR, K = 64 samples)   A = E, B = S (LDS)
// P is formed transposed because its result layout (lane l: samples
// 4 (l / 16) + j, row l % 16) is GEMM2's A operand when K step j of a
// 16-sample tile takes samples 4 k + j: E never leaves the registers.  Rows
// of S move straight from memory to LDS, one chunk ahead and double buffered;
// a chunk's fibers are requested during the previous chunk's GEMM2 (the first
// one's during its own GEMM1), its indices two chunks ahead.
//
// Operand layouts of v_mfma_f32_16x16x4_f32 (one wavefront, lane l):
//   A: A[l % 16][l / 16]   B: B[l / 16][l % 16]   D: D[4 (l / 16) + j][l % 16], j < 4.
//
// Bound: matrix-core time on long groups (every column of a 400^3 tensor,
// ranks 10: 25.6 GFLOP a launch); two blocks per CU cover each other's
// barriers.  That launch takes 331 us (77 TFLOP/s; padding of rows, K and
// columns makes it 97 of the 157 the matrix cores have); 516 us with
// one-float LDS operands, the residual staged through LDS and one block per
// CU.  64 x 64 x 64 x 64, ranks 5, m 512: 7.9 -> 6.9 us.
#include "grad_wide.hpp"

namespace trk {

template <int CT>
struct StreamCfg {
    static constexpr int TF = kGradF32Samples;
    // GEMM2 column tiles: CT in 16-byte reads of 4 tiles and one read of the
    // remaining 1, 2 or 3 (as 4)
    static constexpr int V4 = CT / 4 + (CT % 4 == 3 ? 1 : 0), REM = CT % 4 == 3 ? 0 : CT % 4;
    static constexpr int CW = 4 * V4 + REM;
    static constexpr int Q = 4 * CT + 1, SP = 4 * Q;   // row pitch: an odd number of 16-byte pieces
    static constexpr int NW = (TF - 1) * SP + (16 * CW > 16 * CT ? 16 * CW : 16 * CT);   // words read
    static constexpr int STAGE = (NW + 255) / 256 * 256;                                 // words staged
    static constexpr size_t shm() { return (size_t)2 * STAGE * 4 + (size_t)3 * TF * 20 + 64; }
};

// Direct memory-to-LDS staging of TF rows of S at pitch SP words, BYTES (4 or
// 16) a lane.  A word past R_n R_{n+1} in its row holds some entry of S; rows
// past the last sample hold the last one's.  The words GEMM1 reads there meet
// a zero of G, those GEMM2 reads feed a dropped column or a zero residual.
template <int CT, int BYTES>
__device__ __forceinline__ void stream_stage(const float* __restrict__ S, float* sS, int RR, int f0, int m, int wu,
                                             int l) {
    using C = StreamCfg<CT>;
    constexpr int PW = BYTES / 4, PR = C::SP / PW;   // words and pieces
    constexpr int NI = C::STAGE / (64 * PW);         // wavefront instructions of the block
    const int rp = RR / PW;                          // pieces of a row of S
    int f = (64 * wu + l) / PR, k = (64 * wu + l) - f * PR;
    // opaque: the addresses are formed anew for every chunk instead of being
    // kept across the products in (NI + 3) / 4 registers
    asm volatile("" : "+v"(f), "+v"(k));
#pragma unroll
    for (int i = 0; i < (NI + 3) / 4; ++i) {
        const int c = 4 * i + wu;
        if (c < NI) {   // uniform
            const int fr = f0 + f < m ? f0 + f : m - 1, kc = k < rp ? k : rp - 1;
            const float* src = S + ((int64_t)fr * RR + (int64_t)kc * PW);
            if constexpr (BYTES == 16) __builtin_amdgcn_global_load_lds(src, sS + 64 * PW * c, 16, 0, 0);
            else __builtin_amdgcn_global_load_lds(src, sS + 64 * PW * c, 4, 0, 0);
        }
        k += 256 % PR;
        f += 256 / PR;
        if (k >= PR) {
            k -= PR;
            ++f;
        }
    }
}

template <typename TX, int CT, int BYTES>
__global__ __launch_bounds__(256, CT <= 12 ? 2 : 1) void k_grad_mfma_f32(tr_desc d, ModeSrc ms, Ptrs cores, XSrc xsrc,
                                                          const int32_t* __restrict__ idx,
                                                          const float* __restrict__ S, const double* __restrict__ pF,
                                                          int m, int groups, int row_tiles_max,
                                                          float* __restrict__ gpart, double* __restrict__ lpart,
                                                          int maxIRR, int rr_fixed, WideModes tab) {
    using C = StreamCfg<CT>;
    constexpr int TF = C::TF, SP = C::SP, NU = TF / 16, KQ = 4 * CT;
    int rtile, sgrp;
    if (!xcd_tile_group(row_tiles_max, groups, rtile, sgrp)) return;
    const int N = d.N;
    const int tid = threadIdx.x, l = tid & 63, lr = l & 15, lk = l >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nchunks = (m + TF - 1) / TF;
    const int cpg = (nchunks + groups - 1) / groups;
    const int cbeg = sgrp * cpg, cend = min(nchunks, cbeg + cpg);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float* sS = reinterpret_cast<float*>(smem_raw);            // [2][STAGE]
    double* sL = reinterpret_cast<double*>(sS + 2 * C::STAGE);   // [3][TF]
    int64_t* sB = reinterpret_cast<int64_t*>(sL + 3 * TF);       // [3][TF]
    float* sW = reinterpret_cast<float*>(sB + 3 * TF);           // [3][TF]

    // Indices and probability of sample tid % TF of a chunk (clamped).
    struct Meta {
        int ik[kMaxOrder];
        double pf;
    };
    auto load_meta = [&](int ch, Meta& mt) {
        const int fi = ch * TF + (tid & (TF - 1));
        const int64_t fc = fi < m ? fi : m - 1;
#pragma unroll
        for (int k = 0; k < kMaxOrder; ++k) mt.ik[k] = idx[fc * N + (k < N ? k : N - 1)];
        mt.pf = pF[fc];
    };
    // With one R_n R_{n+1} for every mode the first chunk's loads go out
    // before the step's mode has arrived.
    const bool some = cbeg < cend;
    Meta m0, m1;
    if (some) {
        load_meta(cbeg, m0);
        load_meta(cbeg + 1 < cend ? cbeg + 1 : cbeg, m1);
        if (rr_fixed > 0) stream_stage<CT, BYTES>(S, sS, rr_fixed, cbeg * TF, m, w, l);
    }
    uint64_t t;
    int n;
    resolve_mode(ms, N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);
    const int In = d.I[n];
    const int RR = d.R[n] * d.R[ring_next(n, N)];
    const int i0 = rtile * kMfTI;
    if (i0 >= In) {
        __builtin_amdgcn_s_waitcnt(0);   // no direct load outlives the block
        return;
    }
    if (some && rr_fixed <= 0) stream_stage<CT, BYTES>(S, sS, RR, cbeg * TF, m, w, l);
    const WideMode& wm = tab.md[n];

    // Each sample's fiber offset and weights (zero past the end and for an
    // invalid caller index, which contributes nothing).
    auto put_meta = [&](int ch, const Meta& mt) {
        if (tid < TF) {
            bool ok = ch * TF + tid < m;
            int64_t off = 0;
#pragma unroll
            for (int k = 0; k < kMaxOrder; ++k) {
                if (k >= N) break;
                if (k != n && (mt.ik[k] < 0 || mt.ik[k] >= d.I[k])) ok = false;
                off += (int64_t)mt.ik[k] * wm.xs[k];
            }
            const int at = (ch % 3) * TF + tid;
            sB[at] = ok ? off : 0;
            sW[at] = ok ? (float)(wm.wbase / mt.pf) : 0.f;
            sL[at] = ok ? 1.0 / (2.0 * (double)m * mt.pf) : 0.0;
        }
    };

    // B operand of GEMM1: the lane's row of G; lane group lk owns
    // k = KQ lk + q for its K steps q < KQ, so that four consecutive steps of
    // the A operand are one 16-byte read of a row of S.
    const float* Gn = static_cast<const float*>(cores.p[n]);
    const int row = i0 + 16 * w + lr, rowc = row < In ? row : In - 1;
    const bool live = i0 + 16 * w < In;   // uniform
    float gb[KQ];
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
        const int k = KQ * lk + q;
        gb[q] = Gn[(int64_t)rowc * RR + (k < RR ? k : RR - 1)];
    }
    const TX* X = static_cast<const TX*>(xsrc.rep[n] ? xsrc.rep[n] : xsrc.X);
    const int64_t xrow = (int64_t)rowc * (xsrc.rep[n] ? 1 : d.x_stride[n]);

    // Fiber entries (raw) of the lane's row at its samples of a chunk.
    TX xv[NU][4];
    auto load_fibers = [&](int ch) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) xv[u][j] = X[sB[(ch % 3) * TF + 16 * u + 4 * lk + j] + xrow];
    };

    f32x4 acc2[C::CW];
#pragma unroll
    for (int c = 0; c < C::CW; ++c) acc2[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    double lsum = 0.0;

    if (some) {
        put_meta(cbeg, m0);
        if (cbeg + 1 < cend) put_meta(cbeg + 1, m1);
    }
    __builtin_amdgcn_s_waitcnt(0);   // this wavefront's direct loads have landed
    __syncthreads();
    if (some && live) load_fibers(cbeg);
    // G past R_n R_{n+1} as exact zeros, after the loads have been issued
#pragma unroll
    for (int q = 0; q < KQ; ++q) gb[q] = __uint_as_float(__float_as_uint(gb[q]) & (KQ * lk + q < RR ? ~0u : 0u));

    for (int ch = cbeg; ch < cend; ++ch) {
        const float* Sc = sS + ((ch - cbeg) & 1) * C::STAGE;
        // the next chunk's rows and the one after's indices, in flight during
        // this chunk's products; the next chunk's fibers during GEMM2
        if (ch + 1 < cend)
            stream_stage<CT, BYTES>(S, sS + ((ch + 1 - cbeg) & 1) * C::STAGE, RR, (ch + 1) * TF, m, w, l);
        if (ch + 2 < cend) load_meta(ch + 2, m0);
        if (live) {   // uniform
            __builtin_amdgcn_sched_barrier(0);
            f32x4 p[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) p[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            const float* srow = Sc + lr * SP + KQ * lk;
            float4 ac[NU], an[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) ac[u] = *reinterpret_cast<const float4*>(srow + 16 * u * SP);
            __builtin_amdgcn_sched_group_barrier(0x100, NU, 0);
#pragma unroll
            for (int q = 0; q < CT; ++q) {
                if (q + 1 < CT) {
#pragma unroll
                    for (int u = 0; u < NU; ++u)
                        an[u] = *reinterpret_cast<const float4*>(srow + 16 * u * SP + 4 * (q + 1));
                }
#pragma unroll
                for (int u = 0; u < NU; ++u) p[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[u].x, gb[4 * q], p[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < NU; ++u) p[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[u].y, gb[4 * q + 1], p[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < NU; ++u) p[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[u].z, gb[4 * q + 2], p[u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < NU; ++u) p[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ac[u].w, gb[4 * q + 3], p[u], 0, 0, 0);
                if (q + 1 < CT) __builtin_amdgcn_sched_group_barrier(0x100, NU, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 4 * NU, 0);
                if (q + 1 < CT) {
#pragma unroll
                    for (int u = 0; u < NU; ++u) ac[u] = an[u];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // E = X_F - P, scaled; loss estimate
            float ev[NU][4];
            const int mo = (ch % 3) * TF + 4 * lk;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float wf = sW[mo + 16 * u + j];
                    const float e = row < In && wf != 0.f ? Cvt<TX>::to_f32(xv[u][j]) - p[u][j] : 0.f;
                    lsum += (double)e * (double)e * sL[mo + 16 * u + j];
                    ev[u][j] = -e * wf;
                }
            }
            if (ch + 1 < cend) load_fibers(ch + 1);
            // GEMM2: K step (u, j) takes samples 16 u + 4 lk + j; the lane's
            // columns are 64 h + 4 lr + 0..3 of read h, then 64 V4 + REM lr
            // + 0..REM-1 (16 lanes of a read cover consecutive columns)
            __builtin_amdgcn_sched_barrier(0);
            const float* scol = Sc + 4 * lk * SP;
            float4 bc[C::V4 > 0 ? C::V4 : 1], bn[C::V4 > 0 ? C::V4 : 1];
            float rc[2], rn[2];
            auto read_b = [&](int st, float4* b4, float* br) {
                const float* sr = scol + (16 * (st >> 2) + (st & 3)) * SP;
#pragma unroll
                for (int h = 0; h < C::V4; ++h) b4[h] = *reinterpret_cast<const float4*>(sr + 64 * h + 4 * lr);
                if (C::REM == 1) br[0] = sr[64 * C::V4 + lr];
                if (C::REM == 2) {
                    const float2 v = *reinterpret_cast<const float2*>(sr + 64 * C::V4 + 2 * lr);
                    br[0] = v.x;
                    br[1] = v.y;
                }
            };
            constexpr int NR = C::V4 + (C::REM ? 1 : 0);
            read_b(0, bc, rc);
            __builtin_amdgcn_sched_group_barrier(0x100, NR, 0);
#pragma unroll
            for (int st = 0; st < 4 * NU; ++st) {
                if (st + 1 < 4 * NU) read_b(st + 1, bn, rn);
                const float at = ev[st >> 2][st & 3];
#pragma unroll
                for (int h = 0; h < C::V4; ++h) {
                    acc2[4 * h] = __builtin_amdgcn_mfma_f32_16x16x4f32(at, bc[h].x, acc2[4 * h], 0, 0, 0);
                    acc2[4 * h + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(at, bc[h].y, acc2[4 * h + 1], 0, 0, 0);
                    acc2[4 * h + 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(at, bc[h].z, acc2[4 * h + 2], 0, 0, 0);
                    acc2[4 * h + 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(at, bc[h].w, acc2[4 * h + 3], 0, 0, 0);
                }
#pragma unroll
                for (int c = 0; c < C::REM; ++c)
                    acc2[4 * C::V4 + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(at, rc[c], acc2[4 * C::V4 + c], 0, 0, 0);
                if (st + 1 < 4 * NU) __builtin_amdgcn_sched_group_barrier(0x100, NR, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, C::CW, 0);
#pragma unroll
                for (int h = 0; h < C::V4; ++h) bc[h] = bn[h];
#pragma unroll
                for (int c = 0; c < C::REM; ++c) rc[c] = rn[c];
            }
        }
        if (ch + 2 < cend) put_meta(ch + 2, m0);
        __builtin_amdgcn_s_waitcnt(0);   // this wavefront's direct loads have landed
        __syncthreads();
    }
    float* out = gpart + (int64_t)sgrp * maxIRR;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = i0 + 16 * w + 4 * lk + j;
#pragma unroll
        for (int c = 0; c < C::CW; ++c) {
            const int col = c < 4 * C::V4 ? 64 * (c / 4) + 4 * lr + c % 4 : 64 * C::V4 + C::REM * lr + c - 4 * C::V4;
            if (r < In && col < RR) out[(int64_t)r * RR + col] = acc2[c][j];
        }
    }
    __shared__ double red[4];
    const double ws = wave_sum_dpp(lsum);
    if (l == 0) red[w] = ws;
    __syncthreads();
    if (tid == 0) lpart[(int64_t)sgrp * row_tiles_max + rtile] = ((red[0] + red[1]) + red[2]) + red[3];
}

template <typename TX, int CT>
__global__ __launch_bounds__(256) void k_grad_mfma_f32w(tr_desc d, ModeSrc ms, Ptrs cores, XSrc xsrc,
                                                        const int32_t* __restrict__ idx, const float* __restrict__ S,
                                                        const double* __restrict__ pF, int m, int groups,
                                                        int row_tiles_max, float* __restrict__ gpart,
                                                        double* __restrict__ lpart, int maxIRR, int rr_fixed,
                                                        WideModes tab) {
    grad_f32w_block<TX, CT>((int)blockIdx.x, d, ms, cores, xsrc, idx, S, pF, m, groups, row_tiles_max, gpart, lpart,
                            maxIRR, rr_fixed, tab);
}

template <typename TX, int CT>
static hipError_t launch_wide(const tr_desc& d, ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx, const float* S,
                              const double* pF, int m, dim3 grid, int groups, int row_tiles, float* gp, double* lp,
                              int maxIRR, hipStream_t st) {
    constexpr size_t shm = WideCfg<CT>::shm();
    if (!allow_lds(reinterpret_cast<const void*>(&k_grad_mfma_f32w<TX, CT>), shm)) return hipErrorInvalidValue;
    const WideModes tab = wide_modes(d, xs, m, sizeof(TX));
    launch_timed(k_grad_mfma_f32w<TX, CT>, grid, dim3(256), shm, st, d, ms, cores, xs, idx, S, pF, m, groups,
                 row_tiles, gp, lp, maxIRR, wide_rr_fixed(d), tab);
    return hipGetLastError();
}

template <typename TX>
static hipError_t launch_wide_tx(const tr_desc& d, ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx,
                                 const float* S, const double* pF, int m, dim3 grid, int groups, int row_tiles,
                                 float* gp, double* lp, int maxIRR, int maxRR, hipStream_t st) {
    switch ((maxRR + 15) / 16) {
        case 3: return launch_wide<TX, 3>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR, st);
        case 4: return launch_wide<TX, 4>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR, st);
        case 5: return launch_wide<TX, 5>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR, st);
        case 6: return launch_wide<TX, 6>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR, st);
        case 7: return launch_wide<TX, 7>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR, st);
        case 8: return launch_wide<TX, 8>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR, st);
        default: return hipErrorInvalidValue;
    }
}

template <typename TX, int CT>
static hipError_t launch_stream(const tr_desc& d, ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx, const float* S,
                                const double* pF, int m, dim3 grid, int groups, int row_tiles, float* gp, double* lp,
                                int maxIRR, hipStream_t st) {
    constexpr size_t shm = StreamCfg<CT>::shm();
    // 16-byte pieces of S when every row is whole pieces at an aligned address
    bool wide = (reinterpret_cast<uintptr_t>(S) & 15) == 0;
    for (int k = 0; k < d.N; ++k) wide = wide && (d.R[k] * d.R[(k + 1) % d.N]) % 4 == 0;
    const WideModes tab = wide_modes(d, xs, m, sizeof(TX));
#define TRK_STREAM(BYTES)                                                                                           \
    do {                                                                                                            \
        if (!allow_lds(reinterpret_cast<const void*>(&k_grad_mfma_f32<TX, CT, BYTES>), shm)) return hipErrorInvalidValue; \
        launch_timed(k_grad_mfma_f32<TX, CT, BYTES>, grid, dim3(256), shm, st, d, ms, cores, xs, idx, S, pF, m, groups, \
                     row_tiles, gp, lp, maxIRR, wide_rr_fixed(d), tab);                                             \
    } while (0)
    if (wide) TRK_STREAM(16);
    else TRK_STREAM(4);
#undef TRK_STREAM
    return hipGetLastError();
}

// Smallest compiled tile count covering ceil(maxRR / 16) column tiles.
template <typename TX>
static hipError_t launch_tx(const tr_desc& d, ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx, const float* S,
                            const double* pF, int m, dim3 grid, int groups, int row_tiles, float* gp, double* lp,
                            int maxIRR, int maxRR, hipStream_t st) {
    const int nct = (maxRR + 15) / 16;
#define TRK_CT(C) \
    if (nct <= C) return launch_stream<TX, C>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR, st)
    TRK_CT(1);
    TRK_CT(2);
    TRK_CT(3);
    TRK_CT(4);
    TRK_CT(5);
    TRK_CT(6);
    TRK_CT(7);
    TRK_CT(8);
    TRK_CT(10);
    TRK_CT(12);
    TRK_CT(14);
    TRK_CT(16);
#undef TRK_CT
    return hipErrorInvalidValue;
}

hipError_t launch_grad_mfma_f32(const tr_desc& d, ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx,
                                const float* S, const double* pF, int m, int groups, int row_tiles, float* gp,
                                double* lp, hipStream_t st) {
    const Shape sh = shape_of(d);
    const dim3 grid(xcd_grid(row_tiles, groups));
    const int maxIRR = sh.maxI * sh.maxRR;
    // (the 16-byte form takes one chunk of 128 samples per group whatever
    // chunk the layout chose: with 64-sample chunks m <= 64 groups, and a
    // group past the last sample writes a zero partial)
    if (wide_applies(d, cores, S, gp, m, groups, sh.maxRR, kWideTF)) {
        if (d.x_dtype == TR_F32)
            return launch_wide_tx<float>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR,
                                         sh.maxRR, st);
        if (d.x_dtype == TR_F16)
            return launch_wide_tx<__half>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR,
                                          sh.maxRR, st);
    }
    switch (d.x_dtype) {
        case TR_F32:
            return launch_tx<float>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR,
                                    sh.maxRR, st);
        case TR_F16:
            return launch_tx<__half>(d, ms, cores, xs, idx, S, pF, m, grid, groups, row_tiles, gp, lp, maxIRR,
                                     sh.maxRR, st);
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace trk
