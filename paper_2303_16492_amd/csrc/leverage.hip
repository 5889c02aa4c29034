// a2: the leverage law (Lemma lev_est), in one launch for small cores
// (k_lev_small), else in five; both divide by the rank, which falls below
// min(I_k, R_k R_{k+1}) only on the rank-revealing route.
#include "law.hpp"
#include "sweep.hpp"

namespace trk {

// ----------------------------------------------------- rank-revealing law --
//
// Leverage law of a core whose unfolding may be rank deficient (Lemma
// lev_est divides the scores of Definition "Leverage Scores" by the rank):
// Cholesky with diagonal pivoting on the Gram B = G^T G of G = G_{k(2)}
// (the largest remaining pivot first), stopped once no remaining pivot
// exceeds RR 2^-52 max_i B_ii; r = the steps taken is the rank.  The chosen
// columns P of G span its column space, so with L the r x r factor of B_PP
//     l_i = g_i[P]^T (G_P^T G_P)^{-1} g_i[P] = ||L^{-1} g_i[P]||^2,
// and r = I_k (full row rank, possible only when I_k <= RR) gives l_i = 1.
// One block.  Bm: RR x RR doubles of scratch
// (row-major) holding G^T G on entry, overwritten.  Writes the weights
// floor(l_i / r 2^40) + 1 into w (r = 0, a zero core: the uniform law and
// TR_DEV_ZERO_DIST).
// Pivot test that sends the fast path here: 2^-43 of the largest diagonal
// entry, a few times the rounding of a Gram summed over a few hundred rows
// (so a pivot of a dependent column is caught) while an ill-conditioned core
// of full rank (sigma_min / sigma_max above about 3.4e-7) stays on the fast
// path; both Gram routes carry the same kappa^2 u error on such a core.
constexpr double kLevTrigger = 1.0 / 8796093022208.0;

template <typename TC>
__device__ void leverage_pivoted(const TC* __restrict__ G, int Ik, int RR, double* __restrict__ Bm,
                                 uint64_t* __restrict__ w, int32_t* status) {
    __shared__ int perm[kMaxRR];
    __shared__ double dinv[kMaxRR];
    __shared__ double xw[8][kMaxRR];   // rows are scored by the first eight wavefronts of at least eight
    __shared__ double rv[16];
    __shared__ int ri[16];
    __shared__ double red[16];
    const int tid = threadIdx.x, T = blockDim.x, lane = tid & 63, wid = tid >> 6, nw = T >> 6;
    const int nB = RR;
    for (int i = tid; i < nB; i += T) perm[i] = i;
    __syncthreads();
    double mx = 0.0;
    for (int i = tid; i < nB; i += T) mx = fmax(mx, Bm[(int64_t)i * nB + i]);
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) red[wid] = mx;
    __syncthreads();
    mx = 0.0;
    for (int q = 0; q < nw; ++q) mx = fmax(mx, red[q]);
    const double tol = (double)nB * 2.220446049250313e-16 * mx;
    int r = 0;
    for (int j = 0; j < nB; ++j) {
        // largest remaining pivot (ties: the smallest index)
        double bv = -1.0;
        int bi = nB;
        for (int i = j + tid; i < nB; i += T) {
            const double v = Bm[(int64_t)i * nB + i];
            if (v > bv) { bv = v; bi = i; }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double ov = __shfl_xor(bv, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) { rv[wid] = bv; ri[wid] = bi; }
        __syncthreads();
        bv = rv[0];
        bi = ri[0];
        for (int q = 1; q < nw; ++q)
            if (rv[q] > bv || (rv[q] == bv && ri[q] < bi)) { bv = rv[q]; bi = ri[q]; }
        __syncthreads();
        if (!(bv > tol) || !isfinite(bv)) break;   // the same verdict in every thread
        r = j + 1;
        if (bi != j) {   // symmetric exchange of j and bi: rows (all columns), then columns of the trailing rows
            for (int c = tid; c < nB; c += T) {
                const double a = Bm[(int64_t)j * nB + c];
                Bm[(int64_t)j * nB + c] = Bm[(int64_t)bi * nB + c];
                Bm[(int64_t)bi * nB + c] = a;
            }
            __syncthreads();
            for (int i = j + tid; i < nB; i += T) {
                const double a = Bm[(int64_t)i * nB + j];
                Bm[(int64_t)i * nB + j] = Bm[(int64_t)i * nB + bi];
                Bm[(int64_t)i * nB + bi] = a;
            }
            if (tid == 0) {
                const int a = perm[j];
                perm[j] = perm[bi];
                perm[bi] = a;
            }
            __syncthreads();
        }
        const double ljj = sqrt(Bm[(int64_t)j * nB + j]);
        __syncthreads();
        for (int i = j + 1 + tid; i < nB; i += T) Bm[(int64_t)i * nB + j] /= ljj;
        if (tid == 0) Bm[(int64_t)j * nB + j] = ljj;
        __syncthreads();
        const int wd = nB - j - 1;
        for (int e = tid; e < wd * wd; e += T) {
            const int i = j + 1 + e / wd, c = j + 1 + e % wd;
            Bm[(int64_t)i * nB + c] -= Bm[(int64_t)i * nB + j] * Bm[(int64_t)c * nB + j];
        }
        __syncthreads();
    }
    if (r == 0 || r == Ik) {   // zero core, or full row rank: every score 0 or 1
        if (r == 0 && tid == 0) set_status(status, TR_DEV_ZERO_DIST);
        write_uniform_weights(w, Ik);
        return;
    }
    // L^{-1}: column c by thread c; its diagonal in dinv, the rest in the
    // free upper triangle (entry (jj, c) of L^{-1} at Bm[c][jj]).
    for (int c = tid; c < r; c += T) {
        const double yc = 1.0 / Bm[(int64_t)c * nB + c];
        dinv[c] = yc;
        for (int jj = c + 1; jj < r; ++jj) {
            double acc = Bm[(int64_t)jj * nB + c] * yc;
            for (int k = c + 1; k < jj; ++k) acc += Bm[(int64_t)jj * nB + k] * Bm[(int64_t)c * nB + k];
            Bm[(int64_t)c * nB + jj] = -acc / Bm[(int64_t)jj * nB + jj];
        }
    }
    __syncthreads();
    // l_i, one row per wavefront: x = g_i[P] staged in LDS, then z = L^{-1} x
    // with the lanes over the entries of z.
    double* x = xw[wid & 7];
    for (int i = wid; i < Ik && wid < 8; i += 8) {
        for (int c = lane; c < r; c += 64) x[c] = (double)G[(int64_t)i * RR + perm[c]];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        double acc = 0.0;
        for (int jj = lane; jj < r; jj += 64) {
            double z = dinv[jj] * x[jj];
            for (int c = 0; c < jj; ++c) z += Bm[(int64_t)c * nB + jj] * x[c];
            acc += z * z;
        }
        acc = wave_sum(acc);
        if (lane == 0) w[i] = quantize(acc / (double)r);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    __syncthreads();
}

// G^T G of the whole core (the rank-revealing route of a wide core, whose fast
// test needs only G G^T): every ``units``-th of its lower 16 x 16 tiles from
// ``unit``, by one wavefront on the FP64 matrix cores, both triangles written.
// Ranks 16, 256 x 256 deficient, FP32, whole law: 13.0 ms with one serial sum per
// entry by one workgroup, 11.1 so; 64 x 256 (one launch) 3.6, 2.8 ms.
template <typename TC>
__device__ __forceinline__ void gram_wave_tiles(const TC* __restrict__ G, int Ik, int RR, double* __restrict__ Bm,
                                                int unit, int units) {
    const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
    const int nt = (RR + 15) >> 4, T = nt * (nt + 1) / 2;
    constexpr int U = 8;
    for (int tile = unit; tile < T; tile += units) {   // uniform
        int rt = 0;
        while ((rt + 1) * (rt + 2) / 2 <= tile) ++rt;
        const int r = 16 * rt + lr, c = 16 * (tile - rt * (rt + 1) / 2) + lr;
        const int rc = r < RR ? r : RR - 1, cc = c < RR ? c : RR - 1;
        dbl4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int f0 = 0; f0 < Ik; f0 += 4 * U) {
            TC a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int f = f0 + 4 * u + lk, fc = f < Ik ? f : Ik - 1;
                a[u] = G[(int64_t)fc * RR + rc];
                b[u] = G[(int64_t)fc * RR + cc];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = f0 + 4 * u + lk < Ik;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)a[u] : 0.0, in ? (double)b[u] : 0.0, acc, 0, 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = 16 * rt + 4 * j + lk;
            if (row < RR && c <= row) {
                Bm[(int64_t)row * RR + c] = acc[j];
                Bm[(int64_t)c * RR + row] = acc[j];
            }
        }
    }
}

// Leverage law of core k in five launches across the GPU: the
// FP64 Gram of G_{k(2)} (the sampled-Gram kernels on the core's own rows),
// -(G^T G)^{-1} by the one-workgroup sweep, then
//     l_i = g_i^T (G^T G)^{-1} g_i = -g_i . (g_i (-(G^T G)^{-1}))
// for every row on the FP64 matrix cores, then the weights, CDF and
// (inside a step) the counter advance in one block.  A wide core (I_k <=
// R_k R_{k+1}) takes G G^T (I_k x I_k) through the same Gram and sweep, whose
// rank test is all that is needed: with full row rank every score is 1, and
// without it the launch of the scores forms G^T G for the rank-revealing route.

constexpr int kLevRows = 16;

// l_i for 16 rows per block: wavefront w owns output columns 16 n.., n = w,
// w + 4, ... (K = RR <= RB in steps of 4), each lane's partial dot products
// are added across its 16 lanes, then across the four wavefronts in a fixed
// order.  Loads at clamped indices, masked afterwards; up to RB = 128 both
// column blocks' loads are in flight together, above it one block's.
template <typename TC, int RB>
__global__ __launch_bounds__(256) void k_lev_rows(tr_desc d, ModeSrc ms, int use_mode, int k_fixed, Ptrs cores,
                                                  const double* __restrict__ hm, const int* __restrict__ flag,
                                                  double* __restrict__ gram, double* __restrict__ lev) {
    uint64_t t;
    int k = k_fixed;
    if (use_mode) resolve_mode(ms, d.N, &t, &k);
    const int Ik = d.I[k];
    const int RR = d.R[k] * d.R[ring_next(k, d.N)];
    const int r0 = blockIdx.x * kLevRows;
    const TC* G = static_cast<const TC*>(cores.p[k]);
    if (Ik <= RR) {   // wide: no scores; G^T G over G G^T, which the sweep has read
        if (*flag != 0) gram_wave_tiles(G, Ik, RR, gram, (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), (int)gridDim.x * 4);
        return;
    }
    if (r0 >= Ik) return;
    const int tid = threadIdx.x, l = tid & 63, lr = l & 15, lk = l >> 4, w = tid >> 6;
    constexpr int KS = RB / 4, U = RB <= 128 ? RB / 64 : 1;
    const int row = r0 + lr, rowc = row < Ik ? row : Ik - 1;
    TC ga[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int kk = 4 * ks + lk, kc = kk < RR ? kk : RR - 1;
        ga[ks] = TC(0);
        if (4 * ks < RR) ga[ks] = G[(int64_t)rowc * RR + kc];   // uniform
    }
    double part[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int u0 = 0; u0 < RB / 64; u0 += U) {
        if (16 * (w + 4 * u0) >= RR) break;   // uniform
        double hb[U][KS];
        TC gd[U][4];   // G[r0 + 4 j + lk][c], the entries this lane's outputs pair with
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int kk = 4 * ks + lk, kc = kk < RR ? kk : RR - 1;
            if (4 * ks < RR) {   // uniform
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int c = 16 * (w + 4 * (u0 + u)) + lr, cc = c < RR ? c : RR - 1;
                    hb[u][ks] = hm[(int64_t)kc * RR + cc];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = r0 + 4 * j + lk, rc = r < Ik ? r : Ik - 1;
                const int c = 16 * (w + 4 * (u0 + u)) + lr, cc = c < RR ? c : RR - 1;
                gd[u][j] = G[(int64_t)rc * RR + cc];
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = 16 * (w + 4 * (u0 + u)) + lr;
            dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                if (4 * ks < RR) {
                    const int kk = 4 * ks + lk;
                    const double a = (row < Ik && kk < RR) ? (double)ga[ks] : 0.0;
                    const double b = (kk < RR && c < RR) ? hb[u][ks] : 0.0;
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
                }
#pragma unroll
            for (int j = 0; j < 4; ++j) part[j] += c < RR ? (double)gd[u][j] * acc[j] : 0.0;
        }
    }
    __shared__ double sp[4][kLevRows];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        double v = part[j];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);   // the 16 lanes of one row
        if (lr == 0) sp[w][4 * j + lk] = v;
    }
    __syncthreads();
    if (tid < kLevRows && r0 + tid < Ik)
        lev[r0 + tid] = -(((sp[0][tid] + sp[1][tid]) + sp[2][tid]) + sp[3][tid]);
}

// Weights floor(l_i / RR 2^40) + 1 and their CDF (one block).  When the
// sweep found a pivot at or below 2^-43 max_i h_ii (the Gram is singular or
// close to it), the scores come from the rank-revealing route instead (it
// overwrites the Gram ``gram``).
template <typename TC>
__global__ __launch_bounds__(1024) void k_lev_cdf(tr_desc d, ModeSrc ms, int use_mode, int k_fixed, Ptrs cores,
                                                  double* __restrict__ gram, const double* __restrict__ lev,
                                                  const int* __restrict__ flag, MutPtrs cdf_out, int32_t* status,
                                                  uint64_t* bump, int lds_rows) {
    uint64_t t;
    int k = k_fixed;
    if (use_mode) resolve_mode(ms, d.N, &t, &k);
    const int Ik = d.I[k];
    const int RR = d.R[k] * d.R[ring_next(k, d.N)];
    uint64_t* cdf = static_cast<uint64_t*>(cdf_out.p[k]);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    uint64_t* w = Ik <= lds_rows ? reinterpret_cast<uint64_t*>(smem_raw) : cdf;
    if (*flag != 0) {
        const TC* G = static_cast<const TC*>(cores.p[k]);
        leverage_pivoted(G, Ik, RR, gram, w, status);
    } else if (Ik <= RR) {
        write_uniform_weights(w, Ik);
    } else {
        for (int i = threadIdx.x; i < Ik; i += blockDim.x) w[i] = quantize(lev[i] / (double)RR);
        __syncthreads();
    }
    finish_cdf(w, cdf, Ik, bump);
}

struct LevWs {
    GramWs g;
    size_t gram_off, upd_off, lev_off, total;
    UpdWs u;
};

static LevWs lev_ws_layout(const tr_desc& d) {
    const Shape sh = shape_of(d);
    LevWs L{};
    L.g = gram_ws_layout(d, sh.maxI);
    L.gram_off = L.g.total;
    L.upd_off = L.gram_off + align_up((size_t)sh.maxRR * sh.maxRR * 8);
    L.u = UpdWs{};
    L.u.L_off = 0;
    L.u.flag_off = align_up((size_t)sh.maxRR * sh.maxRR * 8);
    L.u.total = L.u.flag_off + 256;
    L.lev_off = L.upd_off + L.u.total;
    L.total = L.lev_off + align_up((size_t)sh.maxI * 8);
    return L;
}

size_t lev_ws_bytes(const tr_desc& d) { return lev_ws_layout(d).total; }

// ------------------------------------------------------- one-launch form --
//
// The whole law of one core in one workgroup, all of it in LDS: the Gram (of
// columns, or of rows for a wide core) on the FP64 matrix cores, the sweep
// with its rank test by four of the eight wavefronts, the scores, weights and
// CDF.  NT tile columns hold D = min(I_k, R_k R_{k+1}) <= 16 NT.
//
// Gram: wavefront w takes tile w mod T of the T lower tiles and every S-th
// batch of eight K steps; the S partial tiles are added in a fixed order.
// Scores: (-(G^T G)^{-1}) G^T by tiles of 16 rows of G; a lane's B operands are
// the very entries that its products are multiplied with.
//
// Bound: one workgroup's dependent phases (5 us of sweep at D = 25, then the
// Gram's FP64 products).  64^4, ranks 5, FP32, per refresh of one core: five
// launches of 25 us in all (and four gaps), 11.4 so.
constexpr int kLevSmallThreads = 512;
constexpr size_t kLevSmallLds = 100 * 1024;   // with some 40 KB of static LDS: the workgroup has its CU alone

template <typename TC, int NT>
__global__ __launch_bounds__(kLevSmallThreads) void k_lev_small(tr_desc d, ModeSrc ms, int mode_src, int k_fixed,
                                                                Ptrs cores, double* __restrict__ wide_gram,
                                                                size_t wide_stride, MutPtrs cdf_out, int32_t* status,
                                                                uint64_t* bump) {
    uint64_t t;
    int k = mode_src == kLawEveryMode ? (int)blockIdx.x : k_fixed;
    if (mode_src == kLawStepMode) resolve_mode(ms, d.N, &t, &k);
    const int Ik = d.I[k], RR = d.R[k] * d.R[ring_next(k, d.N)];
    const bool wide = Ik <= RR;
    const int D = wide ? Ik : RR, K = wide ? RR : Ik;
    const TC* G = static_cast<const TC*>(cores.p[k]);
    uint64_t* cdf = static_cast<uint64_t*>(cdf_out.p[k]);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* gram = reinterpret_cast<double*>(smem_raw);           // D x D
    double* hm = gram + 16 * NT * 16 * NT;                        // -gram^{-1}, D x D
    uint64_t* w = reinterpret_cast<uint64_t*>(hm + 16 * NT * 16 * NT);   // I_k weights
    __shared__ SweepShared sh;
    const int tid = threadIdx.x, l = tid & 63, lr = l & 15, lk = l >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int W = kLevSmallThreads / 64, T = NT * (NT + 1) / 2, S = W / T > 0 ? W / T : 1, TW = (T + W - 1) / W;
    // Gram(c, e) = sum_f a(c, f) a(e, f), entry (c, f) at c cs + f fs
    const int cs = wide ? RR : 1, fs = wide ? 1 : RR;
    constexpr int U = 8;
    const int part = S > 1 ? wv / T : 0;
    dbl4 acc[TW];
    int rt[TW], ct[TW];
#pragma unroll
    for (int q = 0; q < TW; ++q) {
        acc[q] = dbl4{0.0, 0.0, 0.0, 0.0};
        const int tile = S > 1 ? wv % T : wv + W * q;
        rt[q] = 0;
        while ((rt[q] + 1) * (rt[q] + 2) / 2 <= tile) ++rt[q];
        ct[q] = tile - rt[q] * (rt[q] + 1) / 2;
        if ((S > 1 ? part >= S : tile >= T) || 16 * rt[q] >= D) continue;   // uniform
        const int r = 16 * rt[q] + lr, c = 16 * ct[q] + lr;
        const TC* pr = G + (int64_t)(r < D ? r : D - 1) * cs;
        const TC* pc = G + (int64_t)(c < D ? c : D - 1) * cs;
#pragma unroll 1
        for (int f0 = 4 * U * part; f0 < K; f0 += 4 * U * S) {
            TC a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int f = f0 + 4 * u + lk, fc = f < K ? f : K - 1;
                a[u] = pr[(int64_t)fc * fs];
                b[u] = pc[(int64_t)fc * fs];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = f0 + 4 * u + lk < K;
                acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)a[u] : 0.0, in ? (double)b[u] : 0.0, acc[q], 0, 0, 0);
            }
        }
    }
    for (int p = 0; p < S; ++p) {   // partial tiles in order, both triangles
        if (part == p) {
#pragma unroll
            for (int q = 0; q < TW; ++q) {
                if (S == 1 && wv + W * q >= T) continue;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 16 * rt[q] + 4 * j + lk, c = 16 * ct[q] + lr;
                    if (r < D && c <= r) {
                        const double v = p > 0 ? gram[r * D + c] + acc[q][j] : acc[q][j];
                        gram[r * D + c] = v;
                        gram[c * D + r] = v;
                    }
                }
            }
        }
        __syncthreads();
    }
    int ok_at;
    switch (wv) {
        case 0: ok_at = sweep_wave<NT, 0>(gram, D, 0.0, kLevTrigger, hm, sh); break;
        case 1: ok_at = sweep_wave<NT, 1>(gram, D, 0.0, kLevTrigger, hm, sh); break;
        case 2: ok_at = sweep_wave<NT, 2>(gram, D, 0.0, kLevTrigger, hm, sh); break;
        case kFactorWave: ok_at = sweep_wave<NT, kFactorWave>(gram, D, 0.0, kLevTrigger, hm, sh); break;
        default: ok_at = sweep_wave<NT, kSweepWaves>(gram, D, 0.0, kLevTrigger, hm, sh); break;
    }
    __syncthreads();
    if (ok_at < 0) {
        if (wide) {
            double* Bm = wide_gram + (size_t)(mode_src == kLawEveryMode ? k : 0) * wide_stride;
            gram_wave_tiles(G, Ik, RR, Bm, wv, W);
            __syncthreads();
            leverage_pivoted(G, Ik, RR, Bm, w, status);
        } else {
            leverage_pivoted(G, Ik, RR, gram, w, status);
        }
    } else if (wide) {
        write_uniform_weights(w, Ik);
    } else {
        for (int r0 = 16 * wv; r0 < Ik; r0 += 16 * W) {
            const int row = r0 + lr, rc = row < Ik ? row : Ik - 1;
            TC g[4 * NT];
#pragma unroll
            for (int ks = 0; ks < 4 * NT; ++ks) {
                const int c = 4 * ks + lk;
                g[ks] = G[(int64_t)rc * RR + (c < RR ? c : RR - 1)];
            }
#pragma unroll
            for (int ks = 0; ks < 4 * NT; ++ks) g[ks] = 4 * ks + lk < RR ? g[ks] : TC(0);
            double s = 0.0;
#pragma unroll
            for (int ct2 = 0; ct2 < NT; ++ct2) {
                const int c = 16 * ct2 + lr, cc = c < RR ? c : RR - 1;
                dbl4 o = {0.0, 0.0, 0.0, 0.0};   // rows: columns of G, columns: rows of G
#pragma unroll
                for (int ks = 0; ks < 4 * NT; ++ks) {
                    const int f = 4 * ks + lk;
                    o = __builtin_amdgcn_mfma_f64_16x16x4f64(hm[(f < RR ? f : RR - 1) * D + cc], (double)g[ks], o, 0, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) s = __builtin_fma(o[j], (double)g[4 * ct2 + j], s);
            }
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (lk == 0 && row < Ik) w[row] = quantize(-s / (double)RR);
        }
        __syncthreads();
    }
    finish_cdf(w, cdf, Ik, bump);
}

// Tile columns of the one-launch form, 0 where the five launches are taken:
// every core's smaller side within 64, and the phases of the one workgroup
// (Gram and scores, about 6 I_k NT^2 FP64 cycles) shorter than the launches
// and gaps they replace (five steps and the first refresh of three cores, whole
// pass in us, five launches against one: 250 x 200 x 180 ranks 8 389, 315;
// 400 x 200 x 180 ranks 6 FP64 393, 287; past the line 400 x 300 x 200 ranks 7
// 337, 347 and 700 x 300 x 200 ranks 7 350, 406).
static int lev_small_nt(const tr_desc& d) {
    int nt = 1;
    for (int k = 0; k < d.N; ++k) {
        const int RR = d.R[k] * d.R[ring_next(k, d.N)];
        const int D = d.I[k] < RR ? d.I[k] : RR;
        nt = (D + 15) / 16 > nt ? (D + 15) / 16 : nt;
    }
    if (nt > 4) return 0;
    for (int k = 0; k < d.N; ++k)
        if ((int64_t)d.I[k] * nt * nt > 4096) return 0;
    return nt;
}

// One core's law (mode_src kLawCore: core k, kLawStepMode: the step's mode) or
// every core's (kLawEveryMode).
static hipError_t launch_leverage_one(const tr_desc& d, ModeSrc ms, int mode_src, int k, Ptrs cores, MutPtrs out,
                                      int32_t* status, void* ws, hipStream_t st, uint64_t* bump) {
    const bool f64 = d.core_dtype == TR_F64;
    const Shape sh = shape_of(d);
    const LevWs L = lev_ws_layout(d);
    char* w = static_cast<char*>(ws);
    const size_t gram_elems = (size_t)sh.maxRR * sh.maxRR;
    const int nt = lev_small_nt(d);
#define TRK_LEV_SMALL(NT)                                                                                            \
    do {                                                                                                             \
        auto kern = f64 ? &k_lev_small<double, NT> : &k_lev_small<float, NT>;                                        \
        if (!allow_lds(reinterpret_cast<const void*>(kern), kLevSmallLds)) break;                                    \
        hipLaunchKernelGGL(kern, dim3(mode_src == kLawEveryMode ? d.N : 1), dim3(kLevSmallThreads), kLevSmallLds, st, \
                           d, ms, mode_src, k, cores, reinterpret_cast<double*>(w), gram_elems, out, status, bump);  \
        return hipGetLastError();                                                                                    \
    } while (0)
    // every core at once: a rank-revealing scratch of its own for each
    if (nt > 0 && (mode_src != kLawEveryMode || (size_t)d.N * gram_elems * 8 <= L.total)) {
        if (nt == 1) TRK_LEV_SMALL(1);
        else if (nt == 2) TRK_LEV_SMALL(2);
        else if (nt == 3) TRK_LEV_SMALL(3);
        else TRK_LEV_SMALL(4);
    }
#undef TRK_LEV_SMALL
    if (mode_src == kLawEveryMode) {
        for (int q = 0; q < d.N; ++q) {
            const hipError_t e = launch_leverage_one(d, ms, kLawCore, q, cores, out, status, ws, st, bump);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // the mode source of the Gram, the inverse and the scores: the step's
    // mode, or core k
    const int use_mode = mode_src == kLawStepMode;
    const ModeSrc mk = use_mode ? ms : ModeSrc{nullptr, 0, k, 0};
    double* gram = reinterpret_cast<double*>(w + L.gram_off);
    hipError_t e = launch_gram(d, mk, nullptr, nullptr, sh.maxI, gram, w, L.g, st, nullptr, cores);
    if (e != hipSuccess) return e;
    // no status from the inverse and no damping ladder: a pivot at or
    // below 2^-43 of the largest diagonal entry sends the CDF kernel to
    // the rank-revealing route
    e = launch_sweep_inverse(d, mk, gram, 0.0, L.u, w + L.upd_off, nullptr, st, kLevTrigger);
    if (e != hipSuccess) return e;
    const double* hm = reinterpret_cast<const double*>(w + L.upd_off + L.u.L_off);
    const int* flag = reinterpret_cast<const int*>(w + L.upd_off + L.u.flag_off);
    double* lev = reinterpret_cast<double*>(w + L.lev_off);
    // a block a 16 rows of the scores, or a wavefront a tile of a wide core's G^T G
    const int ntr = (sh.maxRR + 15) / 16, gt = (ntr * (ntr + 1) / 2 + 3) / 4, gr = (sh.maxI + kLevRows - 1) / kLevRows;
    bool wide = false;
    for (int q = 0; q < d.N; ++q) wide = wide || d.I[q] <= d.R[q] * d.R[ring_next(q, d.N)];
    const dim3 grid(wide && gt > gr ? gt : gr);
    // the CDF kernel's static LDS (rank-revealing route, about 20 KB)
    // plus the staged weights stay within 64 KB
    const int lds_rows = sh.maxI <= kLevLdsRows ? sh.maxI : 0;
    const size_t lds = (size_t)lds_rows * 8;
#define TRK_LEV_ROWS(TC, RB) \
    hipLaunchKernelGGL((k_lev_rows<TC, RB>), grid, dim3(256), 0, st, d, ms, use_mode, k, cores, hm, flag, gram, lev)
    if (f64) {
        if (sh.maxRR <= 128) TRK_LEV_ROWS(double, 128);
        else TRK_LEV_ROWS(double, 256);
    } else {
        if (sh.maxRR <= 128) TRK_LEV_ROWS(float, 128);
        else TRK_LEV_ROWS(float, 256);
    }
#undef TRK_LEV_ROWS
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (f64)
        hipLaunchKernelGGL(k_lev_cdf<double>, dim3(1), dim3(1024), lds, st, d, ms, use_mode, k, cores, gram, lev, flag,
                           out, status, bump, lds_rows);
    else
        hipLaunchKernelGGL(k_lev_cdf<float>, dim3(1), dim3(1024), lds, st, d, ms, use_mode, k, cores, gram, lev, flag,
                           out, status, bump, lds_rows);
    return hipGetLastError();
}

hipError_t launch_leverage(const tr_desc& d, ModeSrc ms, int mode_src, int k, Ptrs cores, MutPtrs out,
                           int32_t* status, void* ws, hipStream_t st, uint64_t* bump) {
    return launch_leverage_one(d, ms, mode_src, k, cores, out, status, ws, st, bump);
}

}  // namespace trk
