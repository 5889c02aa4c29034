// a1/a3/a4: mode pick, index draws with their probabilities, and the sampled
// rows of the subchain matrix (Algorithm SSDTP).
//
// S[f][r + R_n s] = M_f(s, r) with M_f = G_{n+1}(i_{n+1}) ... G_{n-1}(i_{n-1})
// (the product of slices of the subchain, Section 3.2).
#include "chain.hpp"

namespace trk {

// A block takes SB samples.  Phase 1: one thread per (sample, mode) draws
// the index (the optimal law: one thread per sample draws over J_n); the
// probabilities are multiplied per sample in the order n+1, ..., n-1.  When
// the kernel draws the step's mode itself and the law is one per mode, the
// index draws do not depend on the mode: threads draw for every mode of
// every sample and one more thread draws the mode, all in the same Philox
// instruction stream, instead of one chain after the other; a draw for the
// step's own mode is dropped.
// do_sample == 2 enumerates instead: sample f is column j = f of X_[n]
// (every column once, m = J_n), decoded in the cyclic order, p = 1/J_n.
// Phase 2, FP32 cores: the chain products of every sample's slices on the
// matrix cores (chain.hpp), each wavefront its packs of samples, every slice
// of a group of packs requested before the first product; the last product is
// written straight to S[f][r + R_n s] = M_f(s, r).  No LDS beyond the draws and
// no barrier after them.
// Phase 2, FP64 cores: the N-1 slices of every sample are copied to LDS in one
// batch; the chain products M <- M G_k(i_k) take one output entry per thread at
// a time (consecutive threads, consecutive columns), accumulated with the
// inner index ascending.
//
// Bound: latency (the draws' generator chain, then one round of slice loads).
// FP32 per launch, with the slices copied to LDS and one product per barrier
// before: 64^4, ranks 5, m 512, leverage law 11.7 -> 7.3 us; 400^3,
// ranks 10, m 4096 8.2 -> 7.0 us; 101 x 57 x 83 x 44, ranks 12/11/9/14, m 2048
// 12.3 -> 10.0 us.
constexpr int kSampleBlock = 16;   // samples of a block

// Packs whose slices a wavefront has in flight together (at most 64 registers
// of slices), NM - 1 slices a sample.
constexpr int sample_packs(int NM) {
    const int u = 64 / ((NM - 1) * 4);
    return u >= 4 ? 4 : (u >= 2 ? 2 : 1);
}

template <typename TC, int RB, bool VEC, int NM, typename OT>
__global__ __launch_bounds__(256) void k_sample_subchain(tr_desc d, ModeSrc ms, int m, int SBf, CdfPtrs cdf,
                                                         const uint64_t* __restrict__ cdf_J, int stream_tag,
                                                         Ptrs cores, int32_t* __restrict__ idx, double* __restrict__ pF,
                                                         TC* __restrict__ S, int do_sample, int do_subchain) {
    const int SB = sizeof(TC) == 4 ? kSampleBlock : SBf;
    const int N = d.N, tid = threadIdx.x;
    const int f0 = blockIdx.x * SB;
    const int nb = min(SB, m - f0);
    uint64_t t;
    int n;
    // per-mode laws with the mode drawn here: the draws of every mode beside
    // the mode's draw (thread nb N), one Philox chain per thread
    const bool early_draws = do_sample == 1 && !cdf_J && ms.n == -1;
    static_assert(16 * kMaxOrder + 1 <= 256, "one thread per (sample, mode) and one for the mode");
    int dr_i = 0;
    double dr_p = 0.0;
    if (early_draws) {
        __shared__ int s_mode;
        t = ms.t_dev ? *ms.t_dev : ms.t;
        if (tid <= nb * N) {
            const bool is_mode = tid == nb * N;
            const int fl = tid / N, k = tid - fl * N;
            const uint64_t r = draw_word(ms.seed, t, is_mode ? 0 : (uint64_t)(f0 + fl), is_mode ? 0 : (uint64_t)k,
                                         is_mode ? (uint64_t)TR_STREAM_MODE : (uint64_t)stream_tag);
            if (is_mode) {
                s_mode = (int)mulhi64(r, (uint64_t)N);
            } else {
                const gptr<uint64_t> ck = lane_pick_global<uint64_t>(cdf.p, k);   // k differs across lanes
                const int Ik = lane_pick(d.I, k);
                if (ck) {
                    dr_i = cdf_pick(ck, Ik, r, &dr_p);
                } else {
                    dr_i = (int)mulhi64(r, (uint64_t)Ik);
                    dr_p = 1.0 / (double)Ik;
                }
            }
        }
        __syncthreads();
        n = __builtin_amdgcn_readfirstlane(s_mode);   // uniform: what follows from it stays scalar
    } else {
        resolve_mode(ms, d.N, &t, &n);
    }
    if (ms.n_pub && blockIdx.x == 0 && threadIdx.x == 0) *ms.n_pub = n;
    const int n1 = ring_next(n, N);
    const int Rn = d.R[n], Rn1 = d.R[n1], RR = Rn * Rn1;
    __shared__ int sidx[kSampleBlock * kMaxOrder];
    __shared__ double sp[kSampleBlock * kMaxOrder];   // order of the chain
    __shared__ int sok[kSampleBlock];
    if (do_sample == 2) {
        const int64_t J = J_of(d, n);
        for (int fl = tid; fl < nb; fl += blockDim.x) {
            int64_t j = f0 + fl;
            sp[fl * kMaxOrder] = 1.0 / (double)J;
            for (int q = 0; q < N - 1; ++q) {
                const int k = (n + 1 + q) % N;
                sidx[fl * kMaxOrder + k] = (int)(j % d.I[k]);
                j /= d.I[k];
            }
            sidx[fl * kMaxOrder + n] = -1;
            sok[fl] = 1;
        }
        __syncthreads();
    } else if (do_sample) {
        if (cdf_J) {
            // thread fl draws sample fl's column (rounds of eight probes, see
            // cdf_pick), decoded in 32-bit divisions where J_n allows
            const int64_t J = J_of(d, n);
            for (int fl = tid; fl < nb; fl += blockDim.x) {
                const uint64_t r = draw_word(ms.seed, t, (uint64_t)(f0 + fl), (uint64_t)n, (uint64_t)stream_tag);
                int64_t j = cdf_pick(cdf_J, J, r, &sp[fl * kMaxOrder]);
                const bool narrow = J <= ((int64_t)1 << 32);   // uniform
                int k = n1;
                for (int q = 0; q < N - 1; ++q) {
                    const int64_t quo = narrow ? (int64_t)((uint32_t)j / (uint32_t)d.I[k]) : j / d.I[k];
                    sidx[fl * kMaxOrder + k] = (int)(j - quo * d.I[k]);
                    j = quo;
                    k = ring_next(k, N);
                }
                sidx[fl * kMaxOrder + n] = -1;
                sok[fl] = 1;
            }
        } else if (early_draws) {
            // thread (sample fl, mode k): its draw at chain position q
            if (tid < nb * N) {
                const int fl = tid / N, k = tid - fl * N;
                if (k == n) {
                    sidx[fl * kMaxOrder + n] = -1;
                    sok[fl] = 1;
                } else {
                    sidx[fl * kMaxOrder + k] = dr_i;
                    const int q = k - n - 1;   // position in the chain n+1, ..., n-1
                    sp[fl * kMaxOrder + (q < 0 ? q + N : q)] = dr_p;
                }
            }
        } else {
            for (int w = tid; w < nb * (N - 1); w += blockDim.x) {
                const int fl = w / (N - 1), q = w - fl * (N - 1);
                const int k = (n + 1 + q) % N;
                const uint64_t r = draw_word(ms.seed, t, (uint64_t)(f0 + fl), (uint64_t)k, (uint64_t)stream_tag);
                const gptr<uint64_t> ck = lane_pick_global<uint64_t>(cdf.p, k);   // k differs across lanes
                const int Ik = lane_pick(d.I, k);
                double pk;
                int i;
                if (ck) {
                    i = cdf_pick(ck, Ik, r, &pk);
                } else {
                    i = (int)mulhi64(r, (uint64_t)Ik);
                    pk = 1.0 / (double)Ik;
                }
                sidx[fl * kMaxOrder + k] = i;
                sp[fl * kMaxOrder + q] = pk;
                if (q == 0) {
                    sidx[fl * kMaxOrder + n] = -1;
                    sok[fl] = 1;
                }
            }
        }
        __syncthreads();
    } else {
        for (int fl = tid; fl < nb; fl += blockDim.x) {
            const int64_t f = f0 + fl;
            int ok = 1;
            for (int k = 0; k < N; ++k) {
                const int i = idx[f * N + k];
                sidx[fl * kMaxOrder + k] = i;
                if (k != n && (i < 0 || i >= d.I[k])) ok = 0;
            }
            sok[fl] = ok;   // invalid caller index: the row is NaN, nothing is read
        }
        __syncthreads();
    }
    // The draws and their probabilities go out after the slice loads are in
    // flight: a store issued before them would hold up their first wait.
    auto write_draws = [&]() {
        for (int fl = tid; fl < nb; fl += blockDim.x) {
            const int64_t f = f0 + fl;
            double p;
            if (cdf_J || do_sample == 2) {
                p = sp[fl * kMaxOrder];
            } else {
                p = 1.0;
                for (int q = 0; q < N - 1; ++q) p = p * sp[fl * kMaxOrder + q];
            }
            pF[f] = p;
            for (int k = 0; k < N; ++k) idx[f * N + k] = sidx[fl * kMaxOrder + k];
        }
    };
    if (!do_subchain) {
        if (do_sample) write_draws();
        return;
    }

    if constexpr (sizeof(TC) == 4) {
        // FP32.  Wavefront w takes packs w, w + 4, ... of P samples.
        constexpr int P = 16 / RB, NPK = kSampleBlock / P, PW = (NPK + 3) / 4, UP = sample_packs(NM), U = UP < PW ? UP : PW;
        const ChainLane<RB> L;
        const ChainSlots<NM - 1, VEC> sl(d, n1, N - 1, L);
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        const bool in0 = L.col < Rn1;
        bool wrote = !do_sample;
#pragma unroll 1
        for (int g = 0; g < PW; g += U) {
            chain4 v[U][NM - 1];
            int fl[U], ok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int pk = wv + 4 * (g + u);
                fl[u] = pk * P + L.p;
                // a sample past the end computes on the block's last one; a rejected
                // caller index reads slice 0 and gives a row of NaN
                const int fc = fl[u] < nb ? fl[u] : nb - 1;
                ok[u] = sok[fc];
                int k = n1;
#pragma unroll
                for (int q = 0; q < NM - 1; ++q) {
                    if (q >= N - 1) break;
                    const int i = ok[u] ? sidx[fc * kMaxOrder + k] : 0;
                    const uint32_t len = (uint32_t)(d.R[k] * d.R[ring_next(k, N)]) * (uint32_t)sizeof(TC);
                    v[u][q] = sl.load(cores.p[k], (OT)(uint32_t)i * (OT)len, q);
                    k = ring_next(k, N);
                }
            }
            if (!wrote) write_draws();   // while the loads above are in flight
            wrote = true;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                chain4 T = sl.mask(v[u][0], 0);
                int k = n1;
#pragma unroll
                for (int q = 1; q < NM - 1; ++q) {
                    if (q >= N - 1) break;
                    k = ring_next(k, N);
                    T = chain_mul(sl.mask(v[u][q], q), T, chain4{0.f, 0.f, 0.f, 0.f});
                    if (q + 1 < N - 1) T = chain_mask(T, L, in0, d.R[ring_next(k, N)]);
                }
                if (fl[u] < nb && in0) {   // S(f, r + R_n s) = M_f(s, r), s = the lane's column, r = its rows
                    TC* out = S + (int64_t)(f0 + fl[u]) * RR + Rn * L.col;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (L.on[j] && L.row[j] < Rn) out[L.row[j]] = ok[u] ? T[j] : TC(NAN);
                }
            }
        }
        return;
    } else {
        // chain order n+1, ..., n-1: stage q is mode (n + 1 + q) mod N; its
        // slice starts at soff[q] within a sample's slices
        extern __shared__ __align__(16) unsigned char smem_raw[];
        TC* sl = reinterpret_cast<TC*>(smem_raw);   // slices, then two product buffers
        __shared__ int soff[kMaxOrder + 1];
        if (tid == 0) {
            int o = 0;
            for (int q = 0; q < N - 1; ++q) {
                soff[q] = o;
                const int k = (n + 1 + q) % N;
                o += d.R[k] * d.R[ring_next(k, N)];
            }
            soff[N - 1] = o;
        }
        __syncthreads();
        int mr = 0;   // largest rank: stride of the product buffers
        for (int k = 0; k < N; ++k) mr = max(mr, d.R[k]);
        // FP64.  Slices of every sample, all loads in flight together.  Thread
        // w of a pass owns value w of every sample's slices (its slice q, mode k
        // and offset are the same for all samples), so the loads of the pass
        // are one per sample at a row taken from LDS: the row is clamped to 0
        // for a rejected caller index and the value masked afterwards, so no
        // load sits behind a branch.
        const int per = soff[N - 1];   // slice values per sample
        for (int w0 = 0; w0 < per; w0 += 256) {
            const int w = w0 + tid, wc = w < per ? w : per - 1;
            int q = 0;
            while (q + 1 < N - 1 && wc >= soff[q + 1]) ++q;
            const int k = (n + 1 + q) % N;
            const int len = soff[q + 1] - soff[q], off = wc - soff[q];
            const gptr<TC> src = lane_pick_global<TC>(cores.p, k);   // k differs across lanes
            constexpr int kSB = 16;   // samples per block at most
            int row[kSB];
            bool ok[kSB];
#pragma unroll
            for (int fl = 0; fl < kSB; ++fl) {   // sample indices clamped into the block's own
                const int fc = fl < nb ? fl : nb - 1;
                const int i = sidx[fc * kMaxOrder + k];
                ok[fl] = sok[fc] != 0;
                row[fl] = ok[fl] ? i : 0;
            }
            TC v[kSB];
#pragma unroll
            for (int fl = 0; fl < kSB; ++fl) v[fl] = src[(int64_t)row[fl] * len + off];
            if (w0 == 0 && do_sample) write_draws();   // while the loads above are in flight
#pragma unroll
            for (int fl = 0; fl < kSB; ++fl)
                if (fl < nb && w < per) sl[(size_t)fl * per + w] = ok[fl] ? v[fl] : TC(0);
        }
        __syncthreads();

        // M (R_{n+1} x R_{k+1}, row-major per sample, stride mr^2)
        // through the chain; slice q of sample fl holds (r, c) at
        // sl[fl * per + soff[q] + r + R_k c].  The last product goes to S.
        const size_t P2 = (size_t)mr * mr;
        TC* bufA = sl + (size_t)SB * per;
        TC* bufB = bufA + (size_t)SB * P2;
        if (N == 2) {
            for (int e = tid; e < nb * RR; e += blockDim.x) {
                const int fl = e / RR, w = e - fl * RR;
                const int s = w / Rn, r = w - s * Rn;
                S[(int64_t)(f0 + fl) * RR + w] = sok[fl] ? sl[(size_t)fl * per + s + Rn1 * r] : TC(NAN);
            }
            return;
        }
        const TC* Mc = nullptr;     // current product; null: the first slice
        int cols = d.R[ring_next(n1, N)];
        for (int q = 1; q < N - 1; ++q) {
            const int k = (n + 1 + q) % N, Rk = d.R[k], Rk1 = d.R[ring_next(k, N)];
            const bool last = q == N - 2;   // then Rk1 == R_n
            TC* Mo = (q & 1) ? bufA : bufB;
            for (int e = tid; e < nb * Rn1 * Rk1; e += blockDim.x) {
                const int fl = e / (Rn1 * Rk1), w = e - fl * (Rn1 * Rk1);
                const int s = w / Rk1, c = w - s * Rk1;
                const TC* A = sl + (size_t)fl * per + soff[q];
                TC acc = TC(0);
                for (int r = 0; r < Rk; ++r) {
                    const TC mv = Mc ? Mc[(size_t)fl * P2 + s * cols + r] : sl[(size_t)fl * per + s + Rn1 * r];
                    acc += mv * A[r + Rk * c];
                }
                if (last)
                    S[(int64_t)(f0 + fl) * RR + w] = sok[fl] ? acc : TC(NAN);
                else
                    Mo[(size_t)fl * P2 + s * Rk1 + c] = acc;
            }
            if (!last) __syncthreads();
            Mc = Mo;
            cols = Rk1;
        }
    }
}

// FP64: samples per block, so that the slices of all of them and two product
// buffers fit in 48 KiB of LDS.
static int sample_block(const tr_desc& d, const Shape& sh, size_t* lds) {
    const size_t per = (size_t)(d.N - 1) * sh.maxR * sh.maxR;
    const size_t prod = d.N > 3 ? 2 * (size_t)sh.maxR * sh.maxR : 0;   // product buffers
    int SB = (int)((48 * 1024) / ((per + prod) * sizeof(double)));
    SB = SB < 1 ? 1 : (SB > kSampleBlock ? kSampleBlock : SB);
    *lds = (size_t)SB * (per + prod) * sizeof(double);
    return SB;
}

hipError_t launch_sample_subchain(const tr_desc& d, ModeSrc ms, int m, CdfPtrs cdf,
                                  const uint64_t* cdf_J, int stream_tag, Ptrs cores,
                                  int32_t* idx, double* pF, void* S, bool do_sample,
                                  bool do_subchain, hipStream_t st) {
    return launch_sample_subchain_mode(d, ms, m, cdf, cdf_J, stream_tag, cores, idx, pF, S, do_sample ? 1 : 0,
                                       do_subchain, st);
}

hipError_t launch_sample_subchain_mode(const tr_desc& d, ModeSrc ms, int m, CdfPtrs cdf,
                                       const uint64_t* cdf_J, int stream_tag, Ptrs cores,
                                       int32_t* idx, double* pF, void* S, int sample_mode,
                                       bool do_subchain, hipStream_t st) {
    if (m <= 0) return hipSuccess;
    const Shape sh = shape_of(d);
    if (d.core_dtype == TR_F64) {
        size_t lds = 0;
        const int SB = sample_block(d, sh, &lds);
        hipLaunchKernelGGL((k_sample_subchain<double, 16, false, 3, uint32_t>), dim3((unsigned)((m + SB - 1) / SB)),
                           dim3(256), do_subchain ? lds : 0, st, d, ms, m, SB, cdf, cdf_J, stream_tag, cores, idx, pF,
                           static_cast<double*>(S), sample_mode, (int)do_subchain);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((m + kSampleBlock - 1) / kSampleBlock));
    // 16-byte slice loads need whole pieces at aligned cores; cores of 4 GiB
    // and more need 64-bit offsets (and take the widest order's form)
    bool vec = do_subchain, big = false;
    for (int k = 0; k < d.N; ++k) {
        vec = vec && d.R[k] % 4 == 0 && (reinterpret_cast<uintptr_t>(cores.p[k]) & 15) == 0;
        big = big || (int64_t)d.I[k] * d.R[k] * d.R[ring_next(k, d.N)] >= ((int64_t)1 << 30);
    }
#define TRK_SMP(RB, VEC, NM, OT)                                                                                    \
    hipLaunchKernelGGL((k_sample_subchain<float, RB, VEC, NM, OT>), grid, dim3(256), 0, st, d, ms, m, kSampleBlock, \
                       cdf, cdf_J, stream_tag, cores, idx, pF, static_cast<float*>(S), sample_mode, (int)do_subchain)
#define TRK_SMP_NM(RB, VEC)                                     \
    do {                                                        \
        if (big) TRK_SMP(RB, VEC, kMaxOrder, uint64_t);         \
        else if (d.N <= 3) TRK_SMP(RB, VEC, 3, uint32_t);       \
        else if (d.N <= 5) TRK_SMP(RB, VEC, 5, uint32_t);       \
        else TRK_SMP(RB, VEC, kMaxOrder, uint32_t);             \
    } while (0)
#define TRK_SMP_RB(RB)                   \
    do {                                 \
        if (vec) TRK_SMP_NM(RB, true);   \
        else TRK_SMP_NM(RB, false);      \
    } while (0)
    if (sh.maxR <= 4) TRK_SMP_RB(4);
    else if (sh.maxR <= 8) TRK_SMP_RB(8);
    else TRK_SMP_RB(16);
#undef TRK_SMP_RB
#undef TRK_SMP_NM
#undef TRK_SMP
    return hipGetLastError();
}

}  // namespace trk
