// a2: the sampling laws of Section 3.2 turned into integer-weight CDFs.
//
//   Euclidean (Lemma euc_est): p(i) = ||G_k(:,i,:)||_F^2 / ||G_k||_F^2.
//   Leverage (Lemma lev_est):  p(i) = l_i(G_{k(2)}) / rank, l_i = g_i^T (G^T G)^{-1} g_i
//                              with the FP64 Gram G^T G of G = G_{k(2)} and its
//                              sweep inverse; with I_k <= R_k R_{k+1} the smaller
//                              G G^T instead, whose full rank makes every l_i 1.  A
//                              Gram that is singular or close to it takes the
//                              rank-revealing route (pivoted Cholesky of G^T G,
//                              scores on the chosen columns, divided by the rank
//                              found).
//   Optimal (eq:optimal_prob): q(j) ~ ||X_[n](:,j) - G_{n(2)} s_j|| * ||s_j||
//                              over the J_n columns, FP64.
// Weights w = floor(p 2^40) + 1 and their inclusive prefix sums are exact
// integers: the sampler's choice depends only on them.
#include "law.hpp"

namespace trk {

// Euclidean law of core k in two launches: the row norms ||g_i||^2 across
// the GPU (a wavefront takes four rows, its lanes across the row, coalesced,
// at most four passes of 64 since RR <= 256, then a shuffle sum), then the
// total, weights, CDF and (inside a step) the counter advance in one block.
constexpr int kEucRows = 16;

// Norms of rows i0 to i0 + NR - 1 (NR a power of two) by one wavefront, NP passes
// of 64 columns.
template <int NR, int NP, typename TC>
__device__ __forceinline__ void euc_rows(const TC* __restrict__ G, int Ik, int RR, int i0, double* rn) {
    const int lane = threadIdx.x & 63;
    if (i0 >= Ik) return;
    double s[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int i = i0 + r < Ik ? i0 + r : Ik - 1;
        s[r] = 0.0;
#pragma unroll
        for (int pa = 0; pa < NP; ++pa) {
            const int c = lane + 64 * pa;
            const double v = (double)G[(int64_t)i * RR + (c < RR ? c : RR - 1)];
            s[r] += c < RR ? v * v : 0.0;
        }
    }
    // The tree of wave_sum for all rows at once: a lane keeps half of its rows
    // and hands the other half over at each of the first log2(NR) levels (a
    // full tree per row is 6 exchanges a row, NR + 2 to NR + 5 here).
    int o = 32;
#pragma unroll
    for (int h = NR / 2; h >= 1; h >>= 1, o >>= 1) {
        const bool up = lane & o;
#pragma unroll
        for (int r = 0; r < h; ++r) {
            const double keep = up ? s[r + h] : s[r], give = up ? s[r] : s[r + h];
            s[r] = keep + __shfl_xor(give, o, 64);
        }
    }
#pragma unroll
    for (; o >= 1; o >>= 1) s[0] += __shfl_xor(s[0], o, 64);
    const int r = lane / (64 / NR);
    if (lane % (64 / NR) == 0 && i0 + r < Ik) rn[i0 + r] = s[0];
}

template <typename TC>
__global__ __launch_bounds__(256) void k_euc_rows(tr_desc d, ModeSrc ms, int use_mode, int k_fixed, Ptrs cores,
                                                  double* __restrict__ rn) {
    uint64_t t;
    int k = k_fixed;
    if (use_mode) resolve_mode(ms, d.N, &t, &k);
    euc_rows<4, 4>(static_cast<const TC*>(cores.p[k]), d.I[k], d.R[k] * d.R[ring_next(k, d.N)],
                   blockIdx.x * kEucRows + 4 * (threadIdx.x >> 6), rn);
}

// Total, weights and CDF from the row norms.
__device__ __forceinline__ void euc_cdf_block(const double* rn, uint64_t* w, uint64_t* cdf, int Ik, int32_t* status,
                                              uint64_t* bump) {
    double loc = 0.0;
    for (int i = threadIdx.x; i < Ik; i += blockDim.x) loc += rn[i];
    __shared__ double red[16];
    const double tot = block_sum(loc, red);
    if (!(tot > 0.0) || !isfinite(tot)) {
        if (threadIdx.x == 0) set_status(status, TR_DEV_ZERO_DIST);
        write_uniform_weights(w, Ik);
    } else {
        for (int i = threadIdx.x; i < Ik; i += blockDim.x) w[i] = quantize(rn[i] / tot);
        __syncthreads();
    }
    finish_cdf(w, cdf, Ik, bump);
}

__global__ __launch_bounds__(1024) void k_euc_cdf(tr_desc d, ModeSrc ms, int use_mode, int k_fixed,
                                                  const double* __restrict__ rn, MutPtrs cdf_out, int32_t* status,
                                                  uint64_t* bump, int lds_rows) {
    uint64_t t;
    int k = k_fixed;
    if (use_mode) resolve_mode(ms, d.N, &t, &k);
    const int Ik = d.I[k];
    uint64_t* cdf = static_cast<uint64_t*>(cdf_out.p[k]);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    euc_cdf_block(rn, Ik <= lds_rows ? reinterpret_cast<uint64_t*>(smem_raw) : cdf, cdf, Ik, status, bump);
}

size_t dist_ws_bytes(const tr_desc& d, int law) {
    const Shape sh = shape_of(d);
    if (law == TR_LAW_EUCLID) return align_up((size_t)sh.maxI * 8);   // row norms
    if (law != TR_LAW_LEVERAGE) return 256;
    return lev_ws_bytes(d);
}

// The Euclidean law in one launch: the same row norms (in the same order),
// total, weights and CDF by one block, everything after the loads in LDS.
// Taken when every core's rows are one round of the block: there it saves a
// launch, past it the exchanges of the row sums on one CU cost more than that
// (five refreshes and three first ones per pass, whole pass in us, two launches
// against one: 64^3 ranks 10 186, 173; 128^3 ranks 10 188, 182; 160^3 ranks 5 154, 177).
constexpr int kEucSmallRows = 128;

template <typename TC>
__global__ __launch_bounds__(1024) void k_euc_small(tr_desc d, ModeSrc ms, int mode_src, int k_fixed, Ptrs cores,
                                                    MutPtrs cdf_out, int32_t* status, uint64_t* bump) {
    uint64_t t;
    int k = mode_src == kLawEveryMode ? (int)blockIdx.x : k_fixed;
    if (mode_src == kLawStepMode) resolve_mode(ms, d.N, &t, &k);
    const int Ik = d.I[k], RR = d.R[k] * d.R[ring_next(k, d.N)];
    __shared__ double rn[kEucSmallRows];
    __shared__ uint64_t w[kEucSmallRows];
    const TC* G = static_cast<const TC*>(cores.p[k]);
    const int i0 = 8 * (threadIdx.x >> 6);   // 16 wavefronts, eight rows each, 8 to 32 loads a lane in flight
    if (RR <= 64) euc_rows<8, 1>(G, Ik, RR, i0, rn);
    else if (RR <= 128) euc_rows<8, 2>(G, Ik, RR, i0, rn);
    else euc_rows<8, 4>(G, Ik, RR, i0, rn);
    __syncthreads();
    euc_cdf_block(rn, w, static_cast<uint64_t*>(cdf_out.p[k]), Ik, status, bump);
}

hipError_t launch_dist(const tr_desc& d, ModeSrc ms, int mode_src, int k, int law, Ptrs cores,
                       uint64_t* const* cdf_out, int32_t* status, void* ws, hipStream_t st, uint64_t* bump) {
    MutPtrs out{};
    for (int q = 0; q < d.N; ++q) out.p[q] = cdf_out[q];
    if (law == TR_LAW_LEVERAGE) return launch_leverage(d, ms, mode_src, k, cores, out, status, ws, st, bump);
    if (law != TR_LAW_EUCLID) return hipErrorInvalidValue;
    const bool f64 = d.core_dtype == TR_F64;
    const Shape sh = shape_of(d);
    if (sh.maxI <= kEucSmallRows) {
        const dim3 grid(mode_src == kLawEveryMode ? d.N : 1);
        if (f64)
            hipLaunchKernelGGL(k_euc_small<double>, grid, dim3(1024), 0, st, d, ms, mode_src, k,
                               cores, out, status, bump);
        else
            hipLaunchKernelGGL(k_euc_small<float>, grid, dim3(1024), 0, st, d, ms, mode_src, k,
                               cores, out, status, bump);
        return hipGetLastError();
    }
    const int first = mode_src == kLawEveryMode ? 0 : k, last = mode_src == kLawEveryMode ? d.N : k + 1;
    const int use_mode = mode_src == kLawStepMode;
    const int lds_rows = sh.maxI <= kLdsRows ? sh.maxI : 0;
    const size_t lds = (size_t)lds_rows * 8;
    double* rn = static_cast<double*>(ws);
    const dim3 grid((sh.maxI + kEucRows - 1) / kEucRows);
    for (int q = first; q < last; ++q) {
        if (f64)
            hipLaunchKernelGGL(k_euc_rows<double>, grid, dim3(256), 0, st, d, ms, use_mode, q, cores, rn);
        else
            hipLaunchKernelGGL(k_euc_rows<float>, grid, dim3(256), 0, st, d, ms, use_mode, q, cores, rn);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_euc_cdf, dim3(1), dim3(1024), lds, st, d, ms, use_mode, q, rn, out, status, bump,
                           lds_rows);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// -------------------------------------------------------------- optimal --

constexpr int kOptBlock = 256;

// a_j = ||X_[n](:,j) - G_{n(2)} s_j||_2 * ||s_j||_2 in FP64, one thread per column.
template <typename TC, typename TX>
__global__ __launch_bounds__(kOptBlock) void k_opt_terms(tr_desc d, ModeSrc ms, Ptrs cores, XSrc xs,
                                                        double* __restrict__ a) {
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);   // uniform: its table reads stay scalar
    const int N = d.N;
    const int n1 = ring_next(n, N);
    const int Rn = d.R[n], Rn1 = d.R[n1];
    const int RR = Rn * Rn1;
    const int64_t J = J_of(d, n);
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= J) return;
    int ik[kMaxOrder];
    int64_t rem = j, off = 0;
    {
        int k = n1;
        for (int q = 1; q < N; ++q) {
            ik[k] = (int)(rem % d.I[k]);
            rem /= d.I[k];
            off += (int64_t)ik[k] * d.x_stride[k];
            k = ring_next(k, N);
        }
    }
    // s_j (row-major in (s, r): s_j[r + Rn s] = M(s, r)), M built row by row.
    double sj[kMaxRR];
    for (int s = 0; s < Rn1; ++s) {
        double v[kMaxRank];
        int k = n1;
        {
            const int Rk = d.R[k], Rk1 = d.R[ring_next(k, N)];
            const TC* A = static_cast<const TC*>(cores.p[k]) + (int64_t)ik[k] * Rk * Rk1;
            for (int c = 0; c < Rk1; ++c) v[c] = (double)A[s + Rk * c];
        }
        for (int q = 2; q < N; ++q) {
            k = ring_next(k, N);
            const int Rk = d.R[k], Rk1 = d.R[ring_next(k, N)];
            const TC* A = static_cast<const TC*>(cores.p[k]) + (int64_t)ik[k] * Rk * Rk1;
            double wv[kMaxRank];
            for (int c = 0; c < Rk1; ++c) {
                double acc = 0.0;
                for (int r = 0; r < Rk; ++r) acc += v[r] * (double)A[r + Rk * c];
                wv[c] = acc;
            }
            for (int c = 0; c < Rk1; ++c) v[c] = wv[c];
        }
        for (int r = 0; r < Rn; ++r) sj[r + Rn * s] = v[r];
    }
    double ss = 0.0;
    for (int c = 0; c < RR; ++c) ss += sj[c] * sj[c];
    const TC* Gn = static_cast<const TC*>(cores.p[n]);
    const TX* X = static_cast<const TX*>(xs.X);
    const int64_t xsn = d.x_stride[n];
    double rr = 0.0;
    for (int i = 0; i < d.I[n]; ++i) {
        double pred = 0.0;
        for (int c = 0; c < RR; ++c) pred += (double)Gn[(int64_t)i * RR + c] * sj[c];
        const double r = to_f64(X[off + (int64_t)i * xsn]) - pred;
        rr += r * r;
    }
    a[j] = sqrt(rr) * sqrt(ss);
}

// The same terms read from the mode-major replica of X, where the fiber
// X_[n](:,j) is contiguous at j I_n (columns in the ring order n+1, n+2, ...
// with the first fastest, as above).  A block takes kOptCols consecutive
// columns.  It forms s_j of every column in LDS: the columns share their
// indices past the first but for a few steps, so the product of the slices of
// cores n+2, ..., n-1 is formed once per such step (one thread per row of it)
// and one thread per (column, row s of the chain product) multiplies the row of
// the column's first slice into it; where a block has more than kOptOuter such
// steps (I_{n+1} < 8) or there is no second slice, that thread walks the whole
// chain.  Each wavefront then takes kOptCols / 4 consecutive columns:
// the predictions G_{n(2)} s_j of its 16 columns are 16 x 16 tiles of FP64
// matrix-core products (its fiber entries requested, in the products'
// result layout, before any arithmetic), and the squared residuals of a
// column are added over its rows in a fixed order.  Needs I_n <= 64 Q,
// R_n R_{n+1} <= RM, every rank <= kOptRank and J_n < 2^31.  bs (optional): the
// sum of the block's terms.
//
// Bound: the loads of the slices and of the fibers (45 MB at the size below).
// 50 x 47 x 53 x 45, ranks 5, FP64: 48.5 us with the whole chain walked per
// column (55 slice loads a thread), 35.8 so; with the fibers or the A operands
// requested earlier 38 to 40 (fewer wavefronts per SIMD).
constexpr int kOptCols = 64;
constexpr int kOptRank = 8;                   // every R_k
constexpr int kOptOuter = 9;                  // runs of columns with the same indices past the first

template <typename TC, typename TX, int Q, int RM>
__global__ __launch_bounds__(256) void k_opt_terms_rep(tr_desc d, ModeSrc ms, Ptrs cores, XSrc xs,
                                                       double* __restrict__ a, double* __restrict__ bs) {
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);   // uniform: its table reads stay scalar
    const int N = d.N;
    const int n1 = ring_next(n, N);
    const int Rn = d.R[n], Rn1 = d.R[n1];
    const int RR = Rn * Rn1, In = d.I[n];
    const int64_t J = J_of(d, n);
    const int64_t j0 = (int64_t)blockIdx.x * kOptCols;
    if (j0 >= J) return;   // the whole block
    __shared__ double sS[kOptCols][RM + 1];
    __shared__ double sN[kOptCols];
    __shared__ double sP[kOptOuter][kOptRank][kOptRank];   // product of the slices past the first, per run
    const int tid = threadIdx.x;
    for (int e = tid; e < kOptCols * (RM + 1); e += 256) (&sS[0][0])[e] = 0.0;
    // Row s of the product of the slices of cores k, ..., n-1 at the indices
    // that rem decodes to (in that order, the first fastest), every loop
    // bounded by kOptRank at compile time so that the row stays in registers
    // and a stage's loads issue together.
    auto chain_row = [&](int k, uint32_t rem, int s, double (&v)[kOptRank]) {
        int Rk = d.R[k], Rk1 = d.R[ring_next(k, N)];
        uint32_t ik = rem % (uint32_t)d.I[k];
        rem /= (uint32_t)d.I[k];
        const TC* A = static_cast<const TC*>(cores.p[k]) + ik * Rk * Rk1;
#pragma unroll
        for (int cc = 0; cc < kOptRank; ++cc) v[cc] = cc < Rk1 ? (double)A[s + Rk * cc] : 0.0;
        for (k = ring_next(k, N); k != n; k = ring_next(k, N)) {
            Rk = d.R[k];
            Rk1 = d.R[ring_next(k, N)];
            ik = rem % (uint32_t)d.I[k];
            rem /= (uint32_t)d.I[k];
            A = static_cast<const TC*>(cores.p[k]) + ik * Rk * Rk1;
            double nv[kOptRank];
#pragma unroll
            for (int cc = 0; cc < kOptRank; ++cc) nv[cc] = 0.0;
#pragma unroll
            for (int r = 0; r < kOptRank; ++r) {
                if (r < Rk) {
#pragma unroll
                    for (int cc = 0; cc < kOptRank; ++cc)
                        if (cc < Rk1) nv[cc] += v[r] * (double)A[r + Rk * cc];
                }
            }
#pragma unroll
            for (int cc = 0; cc < kOptRank; ++cc) v[cc] = nv[cc];
        }
    };
    const int n2 = ring_next(n1, N), Rn2 = d.R[n2];
    const uint32_t I1 = (uint32_t)d.I[n1], jf = (uint32_t)j0, o0 = jf / I1, i10 = jf - o0 * I1;
    const uint32_t jl = (uint32_t)(j0 + kOptCols < J ? j0 + kOptCols : J) - 1;
    const int runs = (int)(jl / I1 - o0) + 1;
    if (N > 2 && runs <= kOptOuter) {   // uniform
        if (tid < runs * Rn2) {
            const int o = tid / Rn2, s = tid - o * Rn2;
            double v[kOptRank];
            chain_row(n2, o0 + o, s, v);
#pragma unroll
            for (int r = 0; r < kOptRank; ++r) sP[o][s][r] = v[r];
        }
        __syncthreads();
        const TC* G1 = static_cast<const TC*>(cores.p[n1]);
        for (int w = tid; w < kOptCols * Rn1; w += 256) {
            const int c = w / Rn1, s = w - c * Rn1;
            if (j0 + c >= J) continue;
            const uint32_t p = i10 + (uint32_t)c, o = p / I1, i1 = p - o * I1;
            const TC* A = G1 + i1 * Rn1 * Rn2;
            TC av[kOptRank];
            double v[kOptRank];
#pragma unroll
            for (int q = 0; q < kOptRank; ++q) av[q] = A[s + Rn1 * (q < Rn2 ? q : 0)];
#pragma unroll
            for (int r = 0; r < kOptRank; ++r) v[r] = 0.0;
#pragma unroll
            for (int q = 0; q < kOptRank; ++q) {
                if (q < Rn2) {
#pragma unroll
                    for (int r = 0; r < kOptRank; ++r) v[r] += (double)av[q] * sP[o][q][r];
                }
            }
#pragma unroll
            for (int r = 0; r < kOptRank; ++r)
                if (r < Rn) sS[c][r + Rn * s] = v[r];
        }
    } else {
        __syncthreads();
        for (int w = tid; w < kOptCols * Rn1; w += 256) {
            const int c = w / Rn1, s = w - c * Rn1;
            if (j0 + c >= J) continue;
            double v[kOptRank];
            chain_row(n1, jf + (uint32_t)c, s, v);
#pragma unroll
            for (int r = 0; r < kOptRank; ++r)
                if (r < Rn) sS[c][r + Rn * s] = v[r];
        }
    }
    // Wavefront w takes the block's columns 16 w .. 16 w + 15.  Its fiber
    // entries are requested before the barrier, in the layout of the matrix
    // core's result: lane l holds column 16 w + l % 16 at rows
    // 16 rt + 4 e + l / 16 (row tile rt, entry e of the 16 x 16 result).
    const int lane = tid & 63, wv = tid >> 6, lc = lane & 15, lk = lane >> 4;
    const int c = wv * 16 + lc;
    const int64_t jc = j0 + c;
    const bool colok = jc < J;
    const TX* Xn = static_cast<const TX*>(xs.rep[n]);
    const int RT = (In + 15) >> 4, KS = (RR + 3) >> 2;
    double xv[4 * Q][4];
#pragma unroll
    for (int rt = 0; rt < 4 * Q; ++rt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * rt + 4 * e + lk;
            xv[rt][e] = (colok && i < In) ? to_f64(Xn[jc * In + i]) : 0.0;
        }
    __syncthreads();
    if (tid < kOptCols) {
        double ss = 0.0;
        for (int cc = 0; cc < RR; ++cc) ss += sS[tid][cc] * sS[tid][cc];
        sN[tid] = ss;
    }
    // pred = G_{n(2)} s_j on the FP64 matrix cores, K = 4 entries of s_j per
    // instruction: A[row][k] = G(16 rt + row, 4 ks + k) (lane l: row l % 16,
    // k = l / 16), B[k][col] = s_j(4 ks + k) of column 16 w + col (lane l:
    // k = l / 16, col = l % 16); entries past R_n R_{n+1} are zeros in sS.
    // (A operands loaded beside the fibers instead measured slower: the
    // extra registers cut the wavefronts per SIMD from 6 to 3.)
    typedef double od4 __attribute__((ext_vector_type(4)));
    const TC* Gn = static_cast<const TC*>(cores.p[n]);
    double bv[RM / 4];
#pragma unroll
    for (int ks = 0; ks < RM / 4; ++ks) bv[ks] = sS[c][4 * ks + lk];
    double rr = 0.0;
#pragma unroll
    for (int rt = 0; rt < 4 * Q; ++rt) {
        if (rt < RT) {
            od4 acc = {0.0, 0.0, 0.0, 0.0};
            const int gi = 16 * rt + lc;
#pragma unroll
            for (int ks = 0; ks < RM / 4; ++ks) {
                if (ks < KS) {
                    const int gk = 4 * ks + lk;
                    const double av = (gi < In && gk < RR) ? (double)Gn[gi * RR + gk] : 0.0;
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[ks], acc, 0, 0, 0);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 16 * rt + 4 * e + lk;
                const double r = xv[rt][e] - acc[e];
                rr += i < In ? r * r : 0.0;
            }
        }
    }
    // the four row groups of each column, in a fixed order
    rr += __shfl_xor(rr, 16, 64);
    rr += __shfl_xor(rr, 32, 64);
    __syncthreads();
    const double term = colok ? sqrt(rr) * sqrt(sN[c]) : 0.0;
    if (lk == 0 && colok) a[jc] = term;
    if (bs) {   // the block's columns in a fixed order: 16 lanes of a wavefront, then the four
        double v = term;
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        __shared__ double sB[4];
        if (lane == 0) sB[wv] = v;
        __syncthreads();
        if (tid == 0) bs[blockIdx.x] = ((sB[0] + sB[1]) + sB[2]) + sB[3];
    }
}

// Per-block FP64 sums of a (fixed order within a block).
__global__ __launch_bounds__(kOptBlock) void k_opt_blocksum(tr_desc d, ModeSrc ms, const double* __restrict__ a,
                                                           double* __restrict__ bs) {
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);   // uniform: its table reads stay scalar
    const int64_t J = J_of(d, n);
    const int64_t nb = (J + kOptBlock - 1) / kOptBlock;
    if (blockIdx.x >= nb) return;
    const int64_t j = (int64_t)blockIdx.x * kOptBlock + threadIdx.x;
    __shared__ double red[kOptBlock / 64];
    const double s = block_sum(j < J ? a[j] : 0.0, red);
    if (threadIdx.x == 0) bs[blockIdx.x] = s;
}

// Total, quantisation, per-block inclusive sums and totals of the weights.
__global__ __launch_bounds__(kOptBlock) void k_opt_quantize(tr_desc d, ModeSrc ms, const double* __restrict__ a,
                                                           const double* __restrict__ bs, int bcols,
                                                           uint64_t* __restrict__ w, uint64_t* __restrict__ wbs,
                                                           int32_t* status) {
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);   // uniform: its table reads stay scalar
    const int64_t J = J_of(d, n);
    const int64_t nb = (J + kOptBlock - 1) / kOptBlock;
    if (blockIdx.x >= nb) return;
    // the total of the sums of bcols columns each, the same fixed order in
    // every block, with the block's own terms in flight beside it
    const int64_t j = (int64_t)blockIdx.x * kOptBlock + threadIdx.x;
    const double aj = a[j < J ? j : J - 1];
    const int64_t ns = (J + bcols - 1) / bcols;
    double part = 0.0;
    for (int64_t b = threadIdx.x; b < ns; b += kOptBlock) part += bs[b];
    __shared__ double red[kOptBlock / 64];
    const double tot = block_sum(part, red);
    const bool zero = !(tot > 0.0) || !isfinite(tot);
    if (zero && blockIdx.x == 0 && threadIdx.x == 0) set_status(status, TR_DEV_ZERO_DIST);
    uint64_t wv = 0;
    if (j < J) wv = zero ? quantize(1.0 / (double)J) : quantize(aj / tot);
    // inclusive scan inside the block: shuffles within a wavefront, then the
    // wavefronts' totals
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up((unsigned long long)wv, (unsigned)o, 64);
        if (lane >= o) wv += y;
    }
    __shared__ uint64_t sc[kOptBlock / 64];
    if (lane == 63) sc[wid] = wv;
    __syncthreads();
    for (int q = 0; q < wid; ++q) wv += sc[q];
    if (j < J) w[j] = wv;
    if (threadIdx.x == kOptBlock - 1) wbs[blockIdx.x] = wv;
}

__global__ __launch_bounds__(1024) void k_opt_offsets(tr_desc d, ModeSrc ms, uint64_t* __restrict__ wbs) {
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);   // uniform: its table reads stay scalar
    const int64_t J = J_of(d, n);
    const int64_t nb = (J + kOptBlock - 1) / kOptBlock;
    // exclusive scan of the block totals, in place: the inclusive scan
    // (integer sums, exact), then every entry takes its predecessor's value,
    // each thread shifting its own segment (the one entry it reads from the
    // segment before is read ahead of a barrier)
    block_scan_u64(wbs, nb);
    const int T = blockDim.x;
    const int64_t per = (nb + T - 1) / T;
    const int64_t b = threadIdx.x * per, e = min(nb, b + per);
    const uint64_t prev = (b > 0 && b < nb) ? wbs[b - 1] : 0ull;
    __syncthreads();
    for (int64_t i = e - 1; i > b; --i) wbs[i] = wbs[i - 1];
    if (b < nb) wbs[b] = prev;
}

// Each block's offset added to its part of the CDF: the sum of the totals
// before it (SUM), or the entry that k_opt_offsets put there.
template <bool SUM>
__global__ __launch_bounds__(kOptBlock) void k_opt_apply(tr_desc d, ModeSrc ms, const uint64_t* __restrict__ wbs,
                                                        uint64_t* __restrict__ w) {
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    n = __builtin_amdgcn_readfirstlane(n);   // uniform: its table reads stay scalar
    const int64_t J = J_of(d, n);
    const int64_t j = (int64_t)blockIdx.x * kOptBlock + threadIdx.x;
    if ((int64_t)blockIdx.x * kOptBlock >= J) return;   // the whole block
    uint64_t off;
    if constexpr (SUM) {
        const uint64_t wj = w[j < J ? j : J - 1];
        unsigned long long part = 0;
        for (int b = threadIdx.x; b < (int)blockIdx.x; b += kOptBlock) part += wbs[b];
        __shared__ unsigned long long red[kOptBlock / 64];
        off = block_sum(part, red);
        if (j < J) w[j] = wj + off;
    } else {
        off = wbs[blockIdx.x];
        if (j < J) w[j] += off;
    }
}

// Up to this many partial sums every block adds them itself (16 loads a thread);
// above it a launch forms the sums of 256 terms or the offsets once.  At
// J = 112 K (441 blocks) the four launches after the terms took 21 us, the two
// left 12.
constexpr int64_t kOptSums = 4096;

size_t dist_opt_ws_bytes(const tr_desc& d) {
    const Shape sh = shape_of(d);
    const int64_t nb = (sh.maxJ + kOptBlock - 1) / kOptBlock;
    // sums: one per block of 256, or one per kOptCols columns
    const int64_t ns = (sh.maxJ + kOptCols - 1) / kOptCols;
    return align_up((size_t)sh.maxJ * 8) + align_up((size_t)(ns <= kOptSums ? ns : nb) * 8) + align_up((size_t)nb * 8);
}

hipError_t launch_dist_optimal(const tr_desc& d, ModeSrc ms, Ptrs cores, XSrc xs, uint64_t* cdf_J, int32_t* status,
                               void* ws, hipStream_t st) {
    const Shape sh = shape_of(d);
    const int64_t nb = (sh.maxJ + kOptBlock - 1) / kOptBlock, ns = (sh.maxJ + kOptCols - 1) / kOptCols;
    char* w = static_cast<char*>(ws);
    double* a = reinterpret_cast<double*>(w);
    double* bs = reinterpret_cast<double*>(w + align_up((size_t)sh.maxJ * 8));
    uint64_t* wbs = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(bs) +
                                                align_up((size_t)(ns <= kOptSums ? ns : nb) * 8));
    const dim3 grid((unsigned)nb);
    const bool f64 = d.core_dtype == TR_F64;
    bool reps = true, summed = false;
    for (int k = 0; k < d.N; ++k) reps = reps && xs.rep[k] != nullptr;
    if (reps && sh.maxI <= 128 && sh.maxR <= kOptRank && sh.maxJ < ((int64_t)1 << 31)) {
        const dim3 gr((unsigned)ns);
        summed = ns <= kOptSums;
        double* sums = summed ? bs : nullptr;
#define TRK_OPT_Q(TC, TX, Q)                                                                                              \
    do {                                                                                                                  \
        if (sh.maxRR <= 32) hipLaunchKernelGGL((k_opt_terms_rep<TC, TX, Q, 32>), gr, dim3(256), 0, st, d, ms, cores, xs, a, sums); \
        else hipLaunchKernelGGL((k_opt_terms_rep<TC, TX, Q, 64>), gr, dim3(256), 0, st, d, ms, cores, xs, a, sums);        \
    } while (0)
#define TRK_OPT(TC, TX)                            \
    do {                                           \
        if (sh.maxI <= 64) TRK_OPT_Q(TC, TX, 1);   \
        else TRK_OPT_Q(TC, TX, 2);                 \
    } while (0)
        if (f64 && d.x_dtype == TR_F64) TRK_OPT(double, double);
        else if (!f64 && d.x_dtype == TR_F32) TRK_OPT(float, float);
        else if (!f64 && d.x_dtype == TR_F16) TRK_OPT(float, __half);
        else return hipErrorInvalidValue;
#undef TRK_OPT
#undef TRK_OPT_Q
    } else if (f64 && d.x_dtype == TR_F64)
        hipLaunchKernelGGL((k_opt_terms<double, double>), grid, dim3(kOptBlock), 0, st, d, ms, cores, xs, a);
    else if (!f64 && d.x_dtype == TR_F32)
        hipLaunchKernelGGL((k_opt_terms<float, float>), grid, dim3(kOptBlock), 0, st, d, ms, cores, xs, a);
    else if (!f64 && d.x_dtype == TR_F16)
        hipLaunchKernelGGL((k_opt_terms<float, __half>), grid, dim3(kOptBlock), 0, st, d, ms, cores, xs, a);
    else
        return hipErrorInvalidValue;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!summed) hipLaunchKernelGGL(k_opt_blocksum, grid, dim3(kOptBlock), 0, st, d, ms, a, bs);
    hipLaunchKernelGGL(k_opt_quantize, grid, dim3(kOptBlock), 0, st, d, ms, a, bs, summed ? kOptCols : kOptBlock, cdf_J, wbs,
                       status);
    if (nb <= kOptSums) {
        hipLaunchKernelGGL(k_opt_apply<true>, grid, dim3(kOptBlock), 0, st, d, ms, wbs, cdf_J);
    } else {
        hipLaunchKernelGGL(k_opt_offsets, dim3(1), dim3(1024), 0, st, d, ms, wbs);
        hipLaunchKernelGGL(k_opt_apply<false>, grid, dim3(kOptBlock), 0, st, d, ms, wbs, cdf_J);
    }
    return hipGetLastError();
}

}  // namespace trk
