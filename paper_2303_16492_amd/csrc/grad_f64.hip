// a5/a6 in FP64: fiber gather, residual and partial gradient on the FP64
// matrix cores (v_mfma_f64_16x16x4f64), prediction first:
// E = X_F - G_{n(2)} S^T, g = -E D S / (m J_n).
//
// A block takes 64 rows of G_{n(2)} (16 per wavefront) and its group's
// samples in chunks of 32, staged in LDS.  A wavefront forms E^T one 16 x 16
// tile at a time (rows: samples, columns: its 16 fiber rows), because
//   - the result layout of that product (lane l, entry j: sample 4 j + l / 16,
//     row l % 16) reads 16 consecutive entries of each fiber, and
//   - it is, entry by entry, the A operand of the second product
//     g[row][c] += E[row][f] S[f][c] at K step j, so E never leaves the
//     registers: no LDS round trip and no barrier between the two products.
// The wavefront's rows of G_{n(2)} stay in registers for all chunks; g is
// accumulated in R_n R_{n+1} / 16 tiles and written once per group.
//
// Bound: latency (indices, then fibers, then two short chains of matrix-core
// steps; 4 I m RR FP64 FLOP is 1.5 us of the chip at 150 x 2000, RR 72).  The
// fibers are requested before the first product needs them.  Measured per
// launch against a vector-unit kernel on 32 x 32 tiles (one LDS read per
// operand per FMA): 150 x 171 x 133, ranks 8/7/9, m 2000: 36.9 -> 13.1 us;
// 50 x 47 x 53 x 45, ranks 5, m 512: 22.0 -> 9.3 us; 20^3, ranks 3, m 100:
// 14.9 -> 8.0 us.
#include "internal.hpp"

namespace trk {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kRows = kGradF64Rows, kTF = kGradF64Samples;

// KB: R_n R_{n+1} <= 16 KB.
template <int KB>
__global__ __launch_bounds__(256, KB <= 8 ? 2 : 1) void k_grad_f64(tr_desc d, ModeSrc ms, Ptrs cores, XSrc xsrc,
                                                                   const int32_t* __restrict__ idx,
                                                                   const double* __restrict__ S,
                                                                   const double* __restrict__ pF, int m, int groups,
                                                                   int row_tiles_max, double* __restrict__ gpart,
                                                                   double* __restrict__ lpart, int maxIRR) {
    int rtile, grp;
    if (!xcd_tile_group(row_tiles_max, groups, rtile, grp)) return;
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);
    const int N = d.N, In = d.I[n];
    const int RR = d.R[n] * d.R[ring_next(n, N)];
    const int i0 = rtile * kRows;
    if (i0 >= In) return;
    const int tid = threadIdx.x, l = tid & 63, lc = l & 15, lk = l >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    extern __shared__ __align__(16) unsigned char smem_raw[];
    // Row pitch 16 ceil(RR / 16) + 2 doubles (twice an odd number): the first
    // product's reads (16 rows, consecutive columns) fall in distinct banks.
    const int W16 = (RR + 15) & ~15, P = W16 + 2;
    double* sS = reinterpret_cast<double*>(smem_raw);   // [kTF][P]
    __shared__ double sW[kTF], sL[kTF], red[4];
    __shared__ int64_t sB[kTF];

    // the source of the fibers: the mode-major replica, or X itself
    const bool rep = xsrc.rep[n] != nullptr;
    const double* X = static_cast<const double*>(rep ? xsrc.rep[n] : xsrc.X);
    const int64_t xsn = rep ? 1 : d.x_stride[n];
    const double Jn = (double)J_of(d, n);
    const double wbase = 1.0 / ((double)m * Jn);

    // the wavefront's 16 rows as the B operand of the first product: lane l
    // holds G(row l % 16, column 4 q + l / 16) for every K step q
    const double* Gn = static_cast<const double*>(cores.p[n]);
    const int gi = i0 + 16 * w + lc;
    const bool live = i0 + 16 * w < In;   // uniform
    double gb[4 * KB];
#pragma unroll
    for (int q = 0; q < 4 * KB; ++q) {
        const int c = 4 * q + lk;
        gb[q] = 0.0;
        if (16 * (q >> 2) < RR)   // uniform
            gb[q] = Gn[(int64_t)(gi < In ? gi : In - 1) * RR + (c < RR ? c : RR - 1)];
    }

    dbl4 acc[KB];
#pragma unroll
    for (int ct = 0; ct < KB; ++ct) acc[ct] = dbl4{0.0, 0.0, 0.0, 0.0};
    double lsum = 0.0;

    const int nchunks = (m + kTF - 1) / kTF;
    const int cpg = (nchunks + groups - 1) / groups;
    const int cbeg = grp * cpg, cend = min(nchunks, cbeg + cpg);
    for (int ch = cbeg; ch < cend; ++ch) {
        const int f0 = ch * kTF;
        // thread (row sr, eighth se) stages columns se + 8 v of sample row sr
        const int sr = tid >> 3, se = tid & 7;
        const double* Srow = S + (int64_t)(f0 + sr < m ? f0 + sr : m - 1) * RR;
        int ik[kMaxOrder];
        double pf = 1.0;
        if (tid < kTF) {
            const int f = f0 + tid < m ? f0 + tid : m - 1;
#pragma unroll
            for (int k = 0; k < kMaxOrder; ++k) ik[k] = idx[(int64_t)f * N + (k < N ? k : N - 1)];
            pf = pF[f];
        }
        double sv[2 * KB];
#pragma unroll
        for (int v = 0; v < 2 * KB; ++v) {
            sv[v] = 0.0;
            if (16 * (v >> 1) < RR) {   // uniform
                const int c = se + 8 * v;
                sv[v] = Srow[c < RR ? c : RR - 1];
            }
        }
        __syncthreads();   // the previous chunk's readers are done
        if (tid < kTF) {
            bool ok = f0 + tid < m;
            int64_t off = 0, st = In;
#pragma unroll
            for (int k = 0; k < kMaxOrder; ++k) {
                if (k >= N || k == n) continue;
                if (ik[k] < 0 || ik[k] >= d.I[k]) ok = false;
                if (!rep) off += (int64_t)ik[k] * d.x_stride[k];
            }
            if (rep) {   // mode-major: mode n fastest, then the ring order after n
#pragma unroll
                for (int k = 0; k < kMaxOrder; ++k)
                    if (k > n && k < N) {
                        off += (int64_t)ik[k] * st;
                        st *= d.I[k];
                    }
#pragma unroll
                for (int k = 0; k < kMaxOrder; ++k)
                    if (k < n) {
                        off += (int64_t)ik[k] * st;
                        st *= d.I[k];
                    }
            }
            // past the end, or an invalid caller index: contributes nothing
            sB[tid] = ok ? off : 0;
            sW[tid] = ok ? wbase / pf : 0.0;
            sL[tid] = ok ? 1.0 / (2.0 * (double)m * pf) : 0.0;
        }
#pragma unroll
        for (int v = 0; v < 2 * KB; ++v) {
            const int c = se + 8 * v;
            if (16 * (v >> 1) < RR) sS[sr * P + c] = c < RR && f0 + sr < m ? sv[v] : 0.0;
        }
        __syncthreads();
        if (!live) continue;   // uniform; the barriers above are met every chunk
        // columns past R_n R_{n+1} as exact zeros (after the barrier, so that
        // no load waits behind the condition)
#pragma unroll
        for (int q = 0; q < 4 * KB; ++q) gb[q] = 4 * q + lk < RR ? gb[q] : 0.0;
        double xv[kTF / 16][4];
#pragma unroll
        for (int ft = 0; ft < kTF / 16; ++ft)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                xv[ft][j] = X[sB[16 * ft + 4 * j + lk] + (int64_t)(gi < In ? gi : In - 1) * xsn];
#pragma unroll
        for (int ft = 0; ft < kTF / 16; ++ft) {
            // E^T tile: A = S (row l % 16, column 4 q + l / 16), B = G^T;
            // two accumulators halve the chain of dependent steps
            dbl4 p0 = {0.0, 0.0, 0.0, 0.0}, p1 = {0.0, 0.0, 0.0, 0.0};
            const double* a = sS + (16 * ft + lc) * P + lk;
#pragma unroll
            for (int qb = 0; qb < KB; ++qb) {
                if (16 * qb < RR) {   // uniform
                    p0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[16 * qb], gb[4 * qb], p0, 0, 0, 0);
                    p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[16 * qb + 4], gb[4 * qb + 1], p1, 0, 0, 0);
                    p0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[16 * qb + 8], gb[4 * qb + 2], p0, 0, 0, 0);
                    p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[16 * qb + 12], gb[4 * qb + 3], p1, 0, 0, 0);
                }
            }
            double ev[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int f = 16 * ft + 4 * j + lk;
                const double wf = sW[f];
                const bool in = gi < In && wf != 0.0;
                const double e = xv[ft][j] - (p0[j] + p1[j]);
                lsum += in ? e * e * sL[f] : 0.0;
                ev[j] = in ? -e * wf : 0.0;
            }
#pragma unroll
            for (int ct = 0; ct < KB; ++ct) {
                if (16 * ct < RR) {   // uniform
                    const double* b = sS + (16 * ft + lk) * P + 16 * ct + lc;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(ev[j], b[4 * j * P], acc[ct], 0, 0, 0);
                }
            }
        }
    }
    double* out = gpart + (int64_t)grp * maxIRR;
    if (live) {
#pragma unroll
        for (int ct = 0; ct < KB; ++ct) {
            if (16 * ct < RR) {   // uniform
                const int c = 16 * ct + lc;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = i0 + 16 * w + 4 * j + lk;
                    if (i < In && c < RR) out[(int64_t)i * RR + c] = acc[ct][j];
                }
            }
        }
    }
    const double tot = block_sum(lsum, red);
    if (tid == 0) lpart[(int64_t)grp * row_tiles_max + rtile] = tot;
}

}  // namespace

hipError_t launch_grad_f64(const tr_desc& d, ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx, const double* S,
                           const double* pF, int m, int groups, int row_tiles, double* gp, double* lp,
                           hipStream_t st) {
    const Shape sh = shape_of(d);
    const dim3 grid(xcd_grid(row_tiles, groups));
    const size_t shm = (size_t)kTF * (((sh.maxRR + 15) & ~15) + 2) * 8;
    const int maxIRR = sh.maxI * sh.maxRR;
#define TRK_GF64(KBV)                                                                                             \
    do {                                                                                                          \
        if (!allow_lds(reinterpret_cast<const void*>(&k_grad_f64<KBV>), shm)) return hipErrorInvalidValue;        \
        launch_timed(k_grad_f64<KBV>, grid, dim3(256), shm, st, d, ms, cores, xs, idx, S, pF, m, groups, row_tiles, \
                     gp, lp, maxIRR);                                                                             \
    } while (0)
    // the register tiles of G and g follow the widest mode
    if (sh.maxRR <= 32) TRK_GF64(2);
    else if (sh.maxRR <= 80) TRK_GF64(5);
    else if (sh.maxRR <= 128) TRK_GF64(8);
    else TRK_GF64(16);
#undef TRK_GF64
    return hipGetLastError();
}

}  // namespace trk
