// a7/a8: the scaled direction p = -g (h + eta I)^{-1}
// (equation eq:scaledsg_direction with the damped preconditioner of the
// remark that follows it), then the step rule.
//
// The RR x RR system is inverted once per step instead of being solved for
// every one of the I_n rows of g: a blocked symmetric sweep (Gauss-Jordan
// elimination on an SPD matrix, eight pivots per block) turns M = h + eta I
// into -M^{-1} in one workgroup, and a second, row-parallel kernel forms
// p = g (-M^{-1}) and applies the rule.  A sweep pivot block is the Schur
// complement of the blocks already swept, so it is positive definite exactly
// when the matching Cholesky pivots are positive: the same test triggers the
// same fallback ladder eta + 10^(k-10) tr(h)/RR, k = 0..6.
//
// The matrix lives in FP64 matrix-core accumulators: 16 x 16 tiles of the
// lower triangle spread over three update wavefronts (tile columns u, 5 - u
// and 6 + u for wavefront u), so each block step moves only the eight pivot
// rows through LDS.  With U~ the pivot columns minus the selector E and
// V~ = U~^T, one block step is the single rank-8 update
//     M <- M - U~ B V~ - 2 E E^T,    B = (M_PP)^{-1},
// which gives -B on the pivot block, B M_PQ on its rows, M_QP B on its
// columns and M_QQ - M_QP B M_PQ elsewhere: the classical sweep.  The
// -2 E E^T term only moves the diagonal of that step's pivot block, which
// no later step reads, so it is applied once at the end.
//
// The fourth wavefront owns no tiles: it works one block ahead.  During
// step q it forms pivot block q+1 as it will be after step q (the Schur
// complement D - C^T B C of the block as published before step q, C the
// pivot rows of step q at its columns, on the vector units) and sweeps that
// 8 x 8 block in registers, so the pivot inverse of every step after the
// first is ready when the step starts.  One barrier per step publishes the next pivot
// rows, the next pivot inverse and its verdict together.
#include "sweep.hpp"

namespace trk {

template <int NT>
__global__ __launch_bounds__(256) void k_sweep(tr_desc d, ModeSrc ms, const double* __restrict__ gram,
                                               Damp dmp, double rank_tol, double* __restrict__ hm,
                                               int* __restrict__ flag, int32_t* status) {
    __shared__ SweepShared sh;
    sweep_block<NT>(d, ms, gram, dmp, rank_tol, hm, flag, status, sh);
}

// ------------------------------------------------ RR in (128, 256] --------
//
// The same sweep for up to 16 tile columns: -(h + eta I)^{-1} of a 132 x 132
// to 256 x 256 system in one workgroup of seven wavefronts.  Six update
// wavefronts share the lower tiles, the seventh (kFactorWave, alone on its
// SIMD) factors the pivot blocks one step ahead exactly as above.
//
// Bound: the chain of RR/8 block steps; a step costs its 2 NT(NT+1)/2 FP64
// matrix-core products over three SIMDs (2.8 K cycles at NT = 11) or the
// factor wavefront's link (2.4 K cycles), whichever is longer.  136 tiles of
// 2 KB exceed the LDS but fit the vector registers of six wavefronts (at most
// 23 tiles of 8 registers each, which at 16 tile columns leaves 15 of the
// other registers in scratch).  Every update wavefront runs the same code
// on tile coordinates held in scalar registers (the per-wavefront code of the
// narrow sweep would be some 150 KB here, past the instruction cache), and
// passes Z = B V~ of its columns to its tiles through its own LDS slots.
//
// Measured (order 4, 101 x 57 x 83 x 44, ranks 12, 11, 9, 14: RR 99 to 168,
// m 2048, Euclidean law, eager): 46 us for the sweep (54 with every slot's
// coordinates compared in every step, see SlotMasks), 116 us per scaled step;
// 749 us with a blocked Cholesky from global memory (475 us) and two triangular
// solves per row (117 us) on one stream.  RR = 256: 192 us with its apply (233).
constexpr int kWideUpd = 6;                         // update wavefronts
constexpr int kWideThreads = 64 * (kWideUpd + 1);
constexpr int kWideCols = 5;   // tile columns a wavefront's run of tiles touches (NT <= 16)

// Column at position p of the order 0, NT-1, 1, NT-2, ... (a tall column next
// to a short one, so that runs of equal length touch few columns).
__host__ __device__ constexpr int wide_col(int p, int NT) { return (p & 1) ? NT - 1 - (p >> 1) : (p >> 1); }
// Tiles of one wavefront for NT tile columns.
__host__ __device__ constexpr int wide_run(int NT) { return (NT * (NT + 1) / 2 + kWideUpd - 1) / kWideUpd; }
// Largest number of columns a run touches.
constexpr int wide_cols_touched(int NT) {
    int worst = 0;
    for (int w = 0; w < kWideUpd; ++w) {
        int at = 0, cols = 0;
        const int s0 = w * wide_run(NT), s1 = s0 + wide_run(NT);
        for (int p = 0; p < NT; ++p) {
            const int h = NT - wide_col(p, NT);
            if (at < s1 && at + h > s0) ++cols;
            at += h;
        }
        worst = cols > worst ? cols : worst;
    }
    return worst;
}
constexpr bool wide_cols_fit() {
    for (int NT = 1; NT <= kMaxRR / 16; ++NT)
        if (wide_cols_touched(NT) > kWideCols) return false;
    return true;
}
static_assert(wide_cols_fit(), "a wavefront's tiles touch at most kWideCols columns");

template <int NTB>
struct WideShared {
    double Vt[2][8 * vt_pitch<NTB>()];
    double Bw[2][40];
    double D8[2][64];
    double Dn[64];
    double zb[kWideUpd][kWideCols][2][64];   // Z of each update wavefront's columns, in operand layout
    double red[kWideUpd + 1];
    double mxdiag;
    int good[2];
};

// Which slots of an update wavefront a block step publishes: lane t holds, for
// tile row t, the slots in it (row), those below its diagonal tile in its
// column (col) and its diagonal tile's slot (diag), so that a step finds its
// slots with three lane reads.  (Comparing every slot's coordinates took some
// 220 cycles a slot and step, half of the wide sweep's step.)
struct SlotMasks {
    int row = 0, col = 0, diag = 0;
    __device__ __forceinline__ void add(int k, int rt, int ct) {
        const int t = threadIdx.x & 15, bit = 1 << k;
        row |= rt == t ? bit : 0;
        col |= ct == t && rt > t ? bit : 0;
        diag |= rt == t && ct == t ? bit : 0;
    }
};

// The tiles of update wavefront uw: slot k is tile (rt, ct) of the wavefront's
// column number m; unused slots have rt = ct = 255 and compute on tile row 15
// and column 0 without being stored or published.  Everything is uniform and
// packed in one scalar register per slot, which every use unpacks anew
// (through an empty asm): addresses and masks derived from it that the
// compiler would keep across the steps took more registers than the tiles.
template <int K>
struct WideTiles {
    int pk[K], cols, n, ncol;   // pk: rt | ct << 8 | m << 16; cols: four bits per column
    SlotMasks M;
    __device__ __forceinline__ static int fresh(int v) {
        asm volatile("" : "+s"(v));
        return v;
    }
    __device__ __forceinline__ void init(int uw, int NT) {
        const int T = NT * (NT + 1) / 2, per = wide_run(NT);
        int s = uw * per, p = 0, at = 0;
        int nn = T - s < per ? T - s : per;
        nn = nn < 0 ? 0 : nn;
        while (p + 1 < NT && at + (NT - wide_col(p, NT)) <= s) {
            at += NT - wide_col(p, NT);
            ++p;
        }
        const int p0 = p;
        int nc = 0, cs = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool in = k < nn;
            const int c = wide_col(p, NT), h = NT - c;
            pk[k] = __builtin_amdgcn_readfirstlane(in ? (c + (s - at)) | c << 8 | (p - p0) << 16 : 0xffff);
            if (in) {
                M.add(k, c + (s - at), c);
                nc = p - p0 + 1;
                cs |= c << (4 * (p - p0));
            }
            ++s;
            if (in && s - at == h) {
                at += h;
                ++p;
            }
        }
        n = __builtin_amdgcn_readfirstlane(nn);
        ncol = __builtin_amdgcn_readfirstlane(nc);
        cols = __builtin_amdgcn_readfirstlane(cs);
    }
};

// One tile's part of the pivot rows (see publish_rows): a tile of the pivot
// tile row, or one of the column below its diagonal tile.
template <int NP, int HQ>
__device__ __forceinline__ void publish_row_tile(const dbl4& a, int ct, int tq, double* Vt) {
    const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
        const double v = a[2 * HQ + jj];
        const int u = 4 * jj + lr, c = 16 * ct + lc;
        // the selector lies in the diagonal tile only: c == 8q + u there is lc == 8 HQ + u
        Vt[u * NP + c] = ct == tq ? v - (lc == 8 * HQ + u ? 1.0 : 0.0) : v;
    }
}
template <int NP, int HQ>
__device__ __forceinline__ void publish_col_tile(const dbl4& a, int rt, double* Vt) {
    const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
    if ((lc >> 3) == HQ) {
#pragma unroll
        for (int j = 0; j < 4; ++j) Vt[(lc - 8 * HQ) * NP + 16 * rt + 4 * j + lr] = a[j];
    }
}

// Slots g to g + 3's part of the pivot rows of block q (row, col: SlotMasks of
// its tile row).
template <int NTB, int K, int HQ>
__device__ __forceinline__ void wide_publish(const dbl4 (&acc)[K], const WideTiles<K>& T, int g, int q, int row, int col,
                                             double* Vt) {
    constexpr int NP = vt_pitch<NTB>();
    if (!((row | col) >> g & 15)) return;
#pragma unroll
    for (int k = g; k < g + 4 && k < K; ++k) {
        if (row >> k & 1) publish_row_tile<NP, HQ>(acc[k], T.fresh(T.pk[k]) >> 8 & 255, q >> 1, Vt);
        else if (col >> k & 1) publish_col_tile<NP, HQ>(acc[k], T.fresh(T.pk[k]) & 255, Vt);
    }
}

// Block step q of an update wavefront (see sweep_step), up to its barrier.
template <int NTB, int K, int HQ>
__device__ __forceinline__ bool wide_update_step(dbl4 (&acc)[K], const WideTiles<K>& T, int uw, WideShared<NTB>& sh,
                                                 int q, int npiv) {
    constexpr int NP = vt_pitch<NTB>();
    const double* Vt = sh.Vt[HQ];
    const double* Bw = sh.Bw[HQ];
    const bool more = q + 1 < npiv;
    const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
    const dbl4 zero = {0.0, 0.0, 0.0, 0.0};
    double a1[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int j = 4 * s + lr;
        const int hi = j > lc ? j : lc, lo = j > lc ? lc : j;
        a1[s] = lc < 8 ? -Bw[tri8(hi & 7) + (lo & 7)] : 0.0;
    }
    double(*zb)[2][64] = sh.zb[uw];
#pragma unroll
    for (int m = 0; m < kWideCols; ++m) {
        if (m < T.ncol) {   // uniform
            const double* v = Vt + 16 * (T.fresh(T.cols) >> (4 * m) & 15) + lc;
            dbl4 z = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[0], v[lr * NP], zero, 0, 0, 0);
            z = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[1], v[(4 + lr) * NP], z, 0, 0, 0);
            zb[m][0][l] = z[0];
            zb[m][1][l] = z[1];
        }
    }
    // this wavefront's LDS stores complete before its own reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // The pivot rows of the next step go out one group of four tiles behind the
    // products, so that the stores run while the matrix cores do.
    int row = 0, col = 0;
    if (more) {
        row = __builtin_amdgcn_readlane(T.M.row, (q + 1) >> 1);
        col = __builtin_amdgcn_readlane(T.M.col, (q + 1) >> 1);
    }
#pragma unroll
    for (int g = 0; g < K + 4; g += 4) {
        if (g < K && g < T.n) {   // uniform; four tiles' operands in flight together
            double u0[4], u1[4], z0[4], z1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (g + i >= K) continue;
                const int pk = T.fresh(T.pk[g + i]), rt = pk & 255, m = pk >> 16;
                const double* u = Vt + lr * NP + 16 * (rt < NTB ? rt : 0) + lc;
                u0[i] = -u[0];
                u1[i] = -u[4 * NP];
                z0[i] = zb[m][0][l];
                z1[i] = zb[m][1][l];
            }
#pragma unroll
            for (int i = 0; i < 4 && g + i < K; ++i)
                acc[g + i] = __builtin_amdgcn_mfma_f64_16x16x4f64(u0[i], z0[i], acc[g + i], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4 && g + i < K; ++i)
                acc[g + i] = __builtin_amdgcn_mfma_f64_16x16x4f64(u1[i], z1[i], acc[g + i], 0, 0, 0);
        }
        if (g > 0) wide_publish<NTB, K, HQ ^ 1>(acc, T, g - 4, q + 1, row, col, sh.Vt[HQ ^ 1]);
    }
    if (q + 2 < npiv) {
        const int diag = __builtin_amdgcn_readlane(T.M.diag, (q + 2) >> 1);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (diag && diag >> k & 1) publish_d8<HQ>(acc[k], sh.D8[HQ]);
    }
    __syncthreads();
    return more ? sh.good[HQ ^ 1] != 0 : true;
}

// The same step of the factor wavefront.
template <int NTB, int HQ>
__device__ __forceinline__ bool wide_factor_step(WideShared<NTB>& sh, int q, int npiv, double tol) {
    const bool more = q + 1 < npiv;
    if (more) {
        const double a = next_pivot_entry<NTB>(sh.Vt[HQ], sh.Bw[HQ], sh.D8[HQ ^ 1], q, sh.Dn);
        const bool g = sweep8_reg(a, sh.Bw[HQ ^ 1], tol);
        if ((threadIdx.x & 63) == 0) sh.good[HQ ^ 1] = g ? 1 : 0;
    }
    __syncthreads();
    return more ? sh.good[HQ ^ 1] != 0 : true;
}

// eta of an attempt of the ladder, tr(h + damping I) / RR found by every
// thread of the block at the second one.
template <int NTB>
__device__ __forceinline__ double wide_eta(const double* __restrict__ gram, int RR, double damping, int attempt,
                                           double& base, WideShared<NTB>& sh) {
    if (attempt == 1) {
        double tr = 0.0;
        for (int c = threadIdx.x; c < RR; c += blockDim.x) tr += gram[(int64_t)c * RR + c];
        base = (block_sum(tr, sh.red) + damping * RR) / RR;
    }
    return attempt == 0 ? damping : damping + pow(10.0, (double)(attempt - 1 - 10)) * base;
}

// Power-of-two scale of the sweep from the largest diagonal entry of
// h + eta I (see sweep_wave).
__device__ __forceinline__ double wide_scale(double mxa) {
    int ex = 0;
    if (!(mxa > 0.0) || !isfinite(mxa)) return 1.0;
    (void)frexp(mxa, &ex);
    return ldexp(1.0, -ex);
}

// The two roles: every barrier of one has its match in the other, and both
// return the attempt that succeeded, or -1.
template <int NTB>
__device__ __forceinline__ int wide_factor_wave(const double* __restrict__ gram, int RR, double damping,
                                                double rank_tol, WideShared<NTB>& sh) {
    const int l = threadIdx.x & 63, npiv = (RR + 7) >> 3;
    double base = 0.0, tol = 0.0, sc = 1.0;
    const int attempts = rank_tol > 0.0 ? 1 : 8;
    for (int attempt = 0; attempt < attempts; ++attempt) {
        const double eta = wide_eta<NTB>(gram, RR, damping, attempt, base, sh);
        // the diagonal and pivot blocks 0 and 1, requested before the barrier
        // and so before the update wavefronts' tiles
        double mx = 0.0, xg[2];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = l + 64 * u, cc = c < RR ? c : RR - 1;
            mx = fmax(mx, gram[(int64_t)cc * RR + cc]);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int r = 8 * b + (l >> 3), c = 8 * b + (l & 7);
            xg[b] = gram[(int64_t)(r < RR ? r : RR - 1) * RR + (c < RR ? c : RR - 1)];
        }
        __syncthreads();   // the previous attempt's readers are done with the shared buffers
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
        if (l == 0) sh.mxdiag = mx;
        __syncthreads();
        if (attempt == 0) {
            sc = wide_scale(mx + eta);
            if (rank_tol > 0.0) tol = rank_tol * (mx + eta) * sc;
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int r = 8 * b + (l >> 3), c = 8 * b + (l & 7);
            const bool in = r < RR && c < RR;
            const double x = in ? (xg[b] + (r == c ? eta : 0.0)) * sc : (r == c ? 1.0 : 0.0);
            if (b == 0) sh.Dn[l] = x;
            else sh.D8[1][l] = x;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const bool g = sweep8(sh.Dn, sh.Bw[0], tol);
        if (l == 0) sh.good[0] = g ? 1 : 0;
        __syncthreads();
        bool good = sh.good[0] != 0;
        for (int q = 0; q < npiv && good; q += 2) {
            good = wide_factor_step<NTB, 0>(sh, q, npiv, tol);
            if (good && q + 1 < npiv) good = wide_factor_step<NTB, 1>(sh, q + 1, npiv, tol);
        }
        if (good) return attempt;
    }
    return -1;
}

template <int NTB, int K>
__device__ __forceinline__ int wide_update_wave(int uw, const double* __restrict__ gram, int RR, double damping,
                                                double rank_tol, double* __restrict__ hm, WideShared<NTB>& sh) {
    const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15, npiv = (RR + 7) >> 3;
    WideTiles<K> T;
    T.init(uw, (RR + 15) >> 4);
    double base = 0.0, sc = 1.0;
    const int attempts = rank_tol > 0.0 ? 1 : 8;
    for (int attempt = 0; attempt < attempts; ++attempt) {
        const double eta = wide_eta<NTB>(gram, RR, damping, attempt, base, sh);
        __syncthreads();   // the previous attempt's readers are done with the shared buffers
        dbl4 acc[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int pk = T.fresh(T.pk[k]), rt = pk & 15, ct = pk >> 8 & 15;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 16 * rt + 4 * j + lr, c = 16 * ct + lc;
                acc[k][j] = gram[(r < RR ? r : RR - 1) * RR + (c < RR ? c : RR - 1)];
            }
        }
        __syncthreads();
        if (attempt == 0) sc = wide_scale(sh.mxdiag + eta);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int pk = T.fresh(T.pk[k]), rt = pk & 255, ct = pk >> 8 & 255;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 16 * rt + 4 * j + lr, c = 16 * ct + lc;
                const bool in = r < RR && c < RR;
                acc[k][j] = in ? (acc[k][j] + (r == c ? eta : 0.0)) * sc : (r == c ? 1.0 : 0.0);
            }
        }
        const int row = __builtin_amdgcn_readlane(T.M.row, 0), col = __builtin_amdgcn_readlane(T.M.col, 0);
#pragma unroll
        for (int g = 0; g < K; g += 4) wide_publish<NTB, K, 0>(acc, T, g, 0, row, col, sh.Vt[0]);
        __syncthreads();
        bool good = sh.good[0] != 0;
        for (int q = 0; q < npiv && good; q += 2) {
            good = wide_update_step<NTB, K, 0>(acc, T, uw, sh, q, npiv);
            if (good && q + 1 < npiv) good = wide_update_step<NTB, K, 1>(acc, T, uw, sh, q + 1, npiv);
        }
        if (good) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int pk = T.fresh(T.pk[k]), rt = pk & 255, ct = pk >> 8 & 255;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 16 * rt + 4 * j + lr, c = 16 * ct + lc;
                    if (r < RR && c < RR) {
                        hm[r * RR + c] = (acc[k][j] - (r == c ? 2.0 : 0.0)) * sc;
                        if (rt != ct) hm[c * RR + r] = acc[k][j] * sc;
                    }
                }
            }
            return attempt;
        }
    }
    return -1;
}

// Contract of k_sweep, for R_n R_{n+1} <= 16 NTB, with K tile slots per
// update wavefront.
template <int NTB, int K>
__global__ __launch_bounds__(kWideThreads) void k_sweep_wide(tr_desc d, ModeSrc ms, const double* __restrict__ gram,
                                                             Damp dmp, double rank_tol, double* __restrict__ hm,
                                                             int* __restrict__ flag, int32_t* status) {
    static_assert(K >= wide_run(NTB), "slots of a wavefront");
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    const double damping = dmp.at(t);
    const int RR = sweep_dim(d, n, rank_tol);
    __shared__ WideShared<NTB> sh;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ok_at = w == kFactorWave
                          ? wide_factor_wave<NTB>(gram, RR, damping, rank_tol, sh)
                          : wide_update_wave<NTB, K>(w < kFactorWave ? w : w - 1, gram, RR, damping, rank_tol, hm, sh);
    if (threadIdx.x == 0) {
        const int fl = ok_at < 0 ? 2 : (ok_at > 0 ? 1 : 0);
        *flag = fl;
        if (fl == 1) set_status(status, TR_DEV_DAMPED);
        if (fl == 2) set_status(status, TR_DEV_NOT_SPD);
    }
}

constexpr int kApplyRows = 16;
constexpr int kApplyWaves = 4;   // the K range split four ways

// p = g (-M^{-1}), then the rule: one 16 x 16 tile of p per block (rows
// 16 blockIdx.x.., columns 16 blockIdx.y..), so the product spreads over
// as many CUs as there are tiles.  Each of the block's four wavefronts runs
// one chain of FP64 matrix-core steps over its quarter of K (K steps of
// four, KW of them: K = R_n R_{n+1} <= 16 KW) on its own SIMD; wavefronts 1-3 leave their
// partial tiles in LDS and wavefront 0 adds them in a fixed order and
// applies the rule.  Every operand (the tile's rows of g, its columns of
// -M^{-1}, the core and accumulator entries it updates) is loaded straight
// from global memory with all loads in flight.  With lp.part set, block
// (0, 0) also writes the loss.  With ``step`` set, the block that finishes
// last advances the step counter (after every block has read it).
// SHAPE0: every mode has the same I_n and R_n R_{n+1}, so the loads of g and
// -M^{-1} are issued before the step's mode has arrived.
template <typename TC, bool SHAPE0, int KW>
__global__ __launch_bounds__(64 * kApplyWaves) void k_scaled_apply(tr_desc d, ModeSrc ms, const TC* __restrict__ g,
                                                                   LossParts lp, double* __restrict__ loss,
                                                                   const double* __restrict__ hm,
                                                                   const int* __restrict__ flag, MutPtrs cores,
                                                                   MutPtrs accum, tr_step rule, int32_t* status,
                                                                   StepBump step) {
    uint64_t t = 0;
    int n = 0;
    if (!SHAPE0) resolve_mode(ms, d.N, &t, &n);
    const int ns = SHAPE0 ? 0 : n;
    const int In = d.I[ns];
    const int RR = d.R[ns] * d.R[ring_next(ns, d.N)];
    const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __shared__ double red[kApplyWaves];
    __shared__ dbl4 part[kApplyWaves - 1][64];
    if (blockIdx.x == 0 && blockIdx.y == 0 && lp.part) {
        const double s = loss_parts_sum(lp, In, red);
        if (threadIdx.x == 0) *loss = s;
    }
    const int r0 = blockIdx.x * kApplyRows, c = 16 * blockIdx.y + lr;
    const bool live = r0 < In && 16 * (int)blockIdx.y < RR;   // uniform
    const int row = r0 + lr, rowc = row < In ? row : In - 1, cc = c < RR ? c : RR - 1;
    dbl4 acc = {0.0, 0.0, 0.0, 0.0};
    TC* G = nullptr;
    TC* A = nullptr;
    double gold[4] = {0.0, 0.0, 0.0, 0.0}, aold[4] = {0.0, 0.0, 0.0, 0.0};
    int fl = 0;
    if (live) {
        // Loads at clamped (in-bounds) indices, masked afterwards: no load
        // sits behind a branch, so all of them are in flight together (with
        // SHAPE0 the ones that do not need the mode go before its read).
        TC ga[KW];
        double hb[KW];
#pragma unroll
        for (int s = 0; s < KW; ++s) {
            const int ks = w * KW + s, k = 4 * ks + lk, kc = k < RR ? k : RR - 1;
            ga[s] = TC(0);
            hb[s] = 0.0;
            if (4 * ks < RR) {   // uniform
                ga[s] = g[(int64_t)rowc * RR + kc];
                hb[s] = hm[(int64_t)kc * RR + cc];
            }
        }
        TC gv[4], av[4];
        if (w == 0) {   // the entries the rule updates
            fl = *flag;
            if (SHAPE0) resolve_mode(ms, d.N, &t, &n);
            G = static_cast<TC*>(cores.p[n]);
            A = static_cast<TC*>(accum.p[n]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = r0 + 4 * j + lk, rc = r < In ? r : In - 1;
                gv[j] = G[(int64_t)rc * RR + cc];
                av[j] = TC(0);
            }
            if (rule.kind == 1) {   // uniform; the accumulator exists only for AdaGrad
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = r0 + 4 * j + lk, rc = r < In ? r : In - 1;
                    av[j] = A[(int64_t)rc * RR + cc];
                }
            }
        }
        double a[KW], b[KW];
#pragma unroll
        for (int s = 0; s < KW; ++s) {
            const int ks = w * KW + s, k = 4 * ks + lk;
            a[s] = (row < In && k < RR) ? (double)ga[s] : 0.0;
            b[s] = (k < RR && c < RR) ? hb[s] : 0.0;
        }
        if (w == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool in = r0 + 4 * j + lk < In && c < RR;
                gold[j] = in ? (double)gv[j] : 0.0;
                aold[j] = in ? (double)av[j] : 0.0;
            }
        }
#pragma unroll
        for (int s = 0; s < KW; ++s)
            if (4 * (w * KW + s) < RR) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
        if (w > 0) part[w - 1][l] = acc;
    }
    __syncthreads();
    if (live && w == 0) {
#pragma unroll
        for (int v = 0; v < kApplyWaves - 1; ++v) acc += part[v][l];   // fixed order
        if (fl != 2) {   // fl == 2: not positive definite even with damping, core unchanged
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = r0 + 4 * j + lk;
                if (r < In && c < RR)
                    apply_rule_loaded<TC>(G, A, (int64_t)r * RR + c, gold[j], aold[j], acc[j], rule, t, status);
            }
        }
    }
    bump_if_last(step, rule.kind == 2);
}

hipError_t launch_sweep_inverse(const tr_desc& d, ModeSrc ms, const double* gram, Damp damping, const UpdWs& L,
                                void* ws, int32_t* status, hipStream_t st, double rank_tol) {
    const Shape sh = shape_of(d);
    char* w = static_cast<char*>(ws);
    double* hm = reinterpret_cast<double*>(w + L.L_off);
    int* flag = reinterpret_cast<int*>(w + L.flag_off);
    const int nt = (sh.maxRR + 15) / 16;
    // The workgroup also reserves the rest of the CU's LDS, which no other
    // workgroup can then share: the sweep is one dependency chain, and
    // waves of a concurrent kernel (the gradient, on the other stream) on
    // its SIMDs would stretch every link of it.
    constexpr size_t kCuLds = 160 * 1024;
#define TRK_SWEEP_K(KERNEL, THREADS, SHARED)                                                                 \
    do {                                                                                                     \
        const size_t reserve = (kCuLds - sizeof(SHARED)) & ~(size_t)1023;                                    \
        const size_t dyn = allow_lds(reinterpret_cast<const void*>(&KERNEL), reserve) ? reserve : 0;         \
        launch_timed(KERNEL, dim3(1), dim3(THREADS), dyn, st, d, ms, gram, damping, rank_tol, hm, flag, status); \
    } while (0)
#define TRK_SWEEP(NTV) TRK_SWEEP_K(k_sweep<NTV>, 256, SweepShared)
#define TRK_SWEEP_WIDE(NTV, KV) TRK_SWEEP_K((k_sweep_wide<NTV, KV>), kWideThreads, WideShared<NTV>)
    // Up to 128 the tiles fit three wavefronts and the narrow sweep, whose
    // tile coordinates are compile-time constants, is the faster one; above
    // it the slots per wavefront (hence its registers) follow the width.
    switch (nt) {
        case 1: TRK_SWEEP(1); break;
        case 2: TRK_SWEEP(2); break;
        case 3: TRK_SWEEP(3); break;
        case 4: TRK_SWEEP(4); break;
        case 5: TRK_SWEEP(5); break;
        case 6: TRK_SWEEP(6); break;
        case 7: TRK_SWEEP(7); break;
        case 8: TRK_SWEEP(8); break;
        case 9:
        case 10:
        case 11: TRK_SWEEP_WIDE(11, 11); break;
        case 12:
        case 13: TRK_SWEEP_WIDE(13, 16); break;
        case 14:
        case 15: TRK_SWEEP_WIDE(15, 20); break;
        default: TRK_SWEEP_WIDE(16, 23); break;
    }
#undef TRK_SWEEP_WIDE
#undef TRK_SWEEP
#undef TRK_SWEEP_K
    return hipGetLastError();
}

hipError_t launch_sweep_apply(const tr_desc& d, ModeSrc ms, const void* g, LossParts lp, double* loss, MutPtrs cores,
                              MutPtrs accum, tr_step rule, int32_t* status, void* ws, const UpdWs& L, StepBump step,
                              hipStream_t st) {
    const Shape sh = shape_of(d);
    char* w = static_cast<char*>(ws);
    const double* hm = reinterpret_cast<const double*>(w + L.L_off);
    const int* flag = reinterpret_cast<const int*>(w + L.flag_off);
    const dim3 grid((sh.maxI + kApplyRows - 1) / kApplyRows, (sh.maxRR + 15) / 16);
    bool same = true;
    for (int k = 1; k < d.N; ++k)
        same = same && d.I[k] == d.I[0] && d.R[k] * d.R[(k + 1) % d.N] == d.R[0] * d.R[1 % d.N];
#define TRK_APPLY_K(TC, S0, KWV)                                                                            \
    hipLaunchKernelGGL((k_scaled_apply<TC, S0, KWV>), grid, dim3(64 * kApplyWaves), 0, st, d, ms, static_cast<const TC*>(g), lp, \
                       loss, hm, flag, cores, accum, rule, status, step)
#define TRK_APPLY(TC, S0)                     \
    do {                                      \
        if (sh.maxRR <= 128) TRK_APPLY_K(TC, S0, 8); \
        else TRK_APPLY_K(TC, S0, 16);         \
    } while (0)
    if (d.core_dtype == TR_F64) {
        if (same) TRK_APPLY(double, true);
        else TRK_APPLY(double, false);
    } else {
        if (same) TRK_APPLY(float, true);
        else TRK_APPLY(float, false);
    }
#undef TRK_APPLY
#undef TRK_APPLY_K
    return hipGetLastError();
}

hipError_t launch_sweep_update(const tr_desc& d, ModeSrc ms, const double* gram, Damp damping, const void* g,
                               double* loss, MutPtrs cores, MutPtrs accum, tr_step rule, int32_t* status, void* ws,
                               const UpdWs& L, StepBump step, hipStream_t st) {
    hipError_t e = launch_sweep_inverse(d, ms, gram, damping, L, ws, status, st);
    if (e != hipSuccess) return e;
    return launch_sweep_apply(d, ms, g, LossParts{}, loss, cores, accum, rule, status, ws, L, step, st);
}

}  // namespace trk
