// a10: sampled-entry loss L = 1/(2B) sum_b (Trace(G_0(i_0^b) ... G_{N-1}(i_{N-1}^b)) - x_b)^2
// and its gradient with respect to every core.
//
// dTrace/dG_k(i_k) = M_{!=k}^T with M_{!=k} = G_{k+1}(i_{k+1}) ...
// G_{k-1}(i_{k-1}), i.e. the row of G^{!=k}_[2] at entry b (the block
// gradient of eq:gradient restricted to sampled entries).
//
// Slice products run on the matrix cores in transposed form, one to four
// entries packed per operand (chain.hpp): a chain needs no LDS.
//
// Forward: a few packs of entries per wavefront; the trace is the sum of T^T S
// over the last slice.  Only the residuals leave the kernel.
//
// Backward: a workgroup owns the gradient slice of one (core, index), or of one
// part of the batch where the mode has few indices.  Each of
// its wavefronts scans its share of the batch's indices of that mode, compacts
// the entries that fall on the slice into an LDS list in entry order, forms
// their M_{!=k} and adds r M_{!=k} by accumulating the chain's last product;
// the wavefronts' sums and the parts are added in a fixed order.  No float atomics: results
// are bitwise reproducible.  (One 4-byte compare per entry and slice is far
// cheaper than private gradient slices per workgroup, whose zeroing, scattered
// read-modify-writes and reduction took most of the time, or than a stable
// sort by index, a serial 26 us per call at B 8192.)
//
// Bound: a chain of dependent memory round trips (indices of the mode, list to
// entry, entry to slices) and instruction issue (operand addresses, masks); the
// products are a few percent.  Measured: order 5, 32 per mode, ranks 8, B 8192:
// forward 13.4 -> 7.3 us (one thread per row of the ring product before),
// backward 40 -> 25 us (private slices); completion, 301 x 250 x 127, ranks
// 10/9/7, B 16384: 35 -> 10 us and 100 -> 30 us, a whole step 169 -> 47 us.
#include <algorithm>
#include <type_traits>

#include "chain.hpp"

namespace trk {

constexpr int kEntBlock = 256;

// loss = 1/(2B) sum of the forward's block partials: strided per thread in
// block order, then the block tree (a fixed order).
__global__ __launch_bounds__(256) void k_entry_loss(const double* __restrict__ part, int nb, int B, double* loss) {
    __shared__ double red[4];
    double s = 0.0;
    for (int q = threadIdx.x; q < nb; q += blockDim.x) s += part[q];
    s = block_sum(s, red);
    if (threadIdx.x == 0) *loss = s / (2.0 * (double)B);
}

typedef chain4 ef4;

// Packs whose slices a wavefront has in flight together: a pack's chain is a
// few hundred cycles of products behind a memory round trip of several times
// that (32 registers of slices).
constexpr int ent_packs(int NM) { return NM <= 3 ? 4 : (NM <= 5 ? 2 : 1); }

// ``iters`` rounds of ent_packs packs per wavefront; NM bounds the order, OT
// holds a byte offset into any core.  Four wavefronts a SIMD up to order 5: without
// whole 16-byte pieces orders 4 and 5 then keep 3 or 4 of their registers in scratch,
// which costs less than the wavefront (60^4, ranks 10, B 16384: 18.7 us; three
// wavefronts and no scratch 21.1).
template <typename TX, int RB, bool VEC, int NM, typename OT>
__global__ __launch_bounds__(kEntBlock, NM <= 5 ? 4 : 2) void k_entry_fwd(tr_desc d, Ptrs cores,
                                                                         const int32_t* __restrict__ idx,
                                                                         const TX* __restrict__ x, int B, int iters,
                                                                         float* __restrict__ resid,
                                                                         double* __restrict__ part) {
    constexpr int P = 16 / RB, U = ent_packs(NM);
    const ChainLane<RB> L;
    const int N = d.N, wv = threadIdx.x >> 6;
    const ChainSlots<NM, VEC> sl(d, 0, N, L);
    const bool in0 = L.col < d.R[0];
    double sq = 0.0;
#pragma unroll 1
    for (int it = 0; it < iters; ++it) {
        const int64_t b0 = (((int64_t)blockIdx.x * iters + it) * (kEntBlock / 64) + wv) * (P * U) + L.p;
        int ik[U][NM];
        float xb[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t b = b0 + P * u, bc = b < B ? b : B - 1;
#pragma unroll
            for (int k = 0; k < NM; ++k)
                if (k < N) ik[u][k] = idx[bc * N + k];
            xb[u] = (float)to_f64(x[bc]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ok[u] = true;
#pragma unroll
            for (int k = 0; k < NM; ++k)
                if (k < N) ok[u] = ok[u] && ik[u][k] >= 0 && ik[u][k] < d.I[k];
        }
        ef4 v[U][NM];
#pragma unroll
        for (int k = 0; k < NM; ++k) {
            if (k >= N) break;
            const int RR = d.R[k] * d.R[ring_next(k, N)];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u][k] = sl.load(cores.p[k], ok[u] ? (OT)ik[u][k] * (OT)(4 * RR) : (OT)0, k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ef4 T = sl.mask(v[u][0], 0);
            float tr = 0.f;
#pragma unroll
            for (int k = 1; k < NM; ++k) {
                if (k >= N) break;
                const ef4 a = sl.mask(v[u][k], k);
                if (k + 1 < N) {
                    T = chain_mask(chain_mul(a, T, ef4{0.f, 0.f, 0.f, 0.f}), L, in0, d.R[ring_next(k, N)]);
                } else {
                    // Trace(T S) = sum over (r, c) of T(r, c) S(c, r) = T^T(c, r) S(c, r)
#pragma unroll
                    for (int j = 0; j < 4; ++j) tr += T[j] * a[j];
                }
            }
            // the lanes of one block, in a fixed order
            tr = L.on[0] ? tr : 0.f;
#pragma unroll
            for (int o = 1; o < RB; o <<= 1) tr += __shfl_xor(tr, o, 64);
            if constexpr (RB >= 8) tr += __shfl_xor(tr, 16, 64);
            if constexpr (RB == 16) tr += __shfl_xor(tr, 32, 64);
            const int64_t b = b0 + P * u;
            if (L.on[0] && L.row[0] == 0 && L.col == 0 && b < B) {
                const float r = ok[u] ? tr - xb[u] : NAN;   // NaN: invalid caller index
                resid[b] = r;
                sq += (double)r * (double)r;
            }
        }
    }
    __shared__ double red[kEntBlock / 64];
    const double tot = block_sum(sq, red);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// The backward's grid: mode k's workgroups start at base[k], ``parts[k]`` of them
// (one a range of the batch) for each of its I_k slices.  at[k]: where the
// partial gradients of a mode of several parts start.
struct EntGroups {
    int64_t base[kMaxOrder + 1], at[kMaxOrder];
    int parts[kMaxOrder];
};
// Wavefronts of a workgroup at most; half of them past order 5, whose seven slices
// in flight take the registers of two.
constexpr int bwd_waves(int NM) { return NM <= 5 ? 16 : 8; }
constexpr int64_t kBwdGrid = 1 << 22;
// Entries of a wavefront's share scanned into its list at a time: at most
// 4096, at least 512 (a 16 x 16 partial tile fits the list's 2-byte places).
constexpr int kBwdWindow = 4096, kBwdWindowMin = 512;

// Part p of gradient slice (k, i) (see the top of the file): the entries of the
// p-th of parts[k] equal ranges of the batch, to grads.p[k] + p I_k R_k R_{k+1}.
// One per workgroup up to a grid of kBwdGrid.  An entry with an invalid index in
// another mode contributes nothing.  The FP32 accumulator covers at most 64 entries
// of the list before it is added to an FP64 total, so the rounding of a slice does
// not grow with the entries that fall on it.
template <int RB, bool VEC, int NM, typename OT>
__global__ __launch_bounds__(64 * bwd_waves(NM)) void k_entry_bwd(tr_desc d, Ptrs cores, const int32_t* __restrict__ idx,
                                                              const float* __restrict__ resid, int B, float scale,
                                                              const double* __restrict__ dscale, EntGroups gr,
                                                              int window, ModeSrc only, int block, MutPtrs grads) {
    constexpr int P = 16 / RB, U = ent_packs(NM), KI = 16;
    extern __shared__ __align__(16) unsigned char smem_raw[];   // [wavefronts][window] 2-byte places
    const ChainLane<RB> L;
    const int N = d.N, tid = threadIdx.x, l = tid & 63, W = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int step_mode = -1;   // block mode: only the step's core moves
    if (block) {
        uint64_t t;
        resolve_mode(only, N, &t, &step_mode);
    }
    int k = 0;
    for (int64_t unit = blockIdx.x; unit < gr.base[N]; unit += gridDim.x) {
        while (k + 1 < N && unit >= gr.base[k + 1]) ++k;
        if (block && step_mode != k) continue;   // uniform
        const int parts = gr.parts[k], at_k = (int)(unit - gr.base[k]);
        const int i = at_k / parts, part = at_k - i * parts, k0 = ring_next(k, N);
        uint16_t* list = reinterpret_cast<uint16_t*>(smem_raw) + w * window;
        // dL/dG_k of L = 1/(2B) sum r^2: the 1/B of the mean applied here
        const float sc = (float)((double)scale * (dscale ? *dscale : 1.0) / (double)B);
        const ChainSlots<NM - 1, VEC> sl(d, k0, N - 1, L);
        const bool in0 = L.col < d.R[k0];
        double tot[4] = {0.0, 0.0, 0.0, 0.0};
        const int64_t share = (((int64_t)B + W * parts - 1) / (W * parts) + 63) & ~63;
        const int64_t s0 = ((int64_t)part * W + w) * share, s1 = min((int64_t)B, s0 + share);
        for (int64_t w0 = s0; w0 < s1; w0 += window) {
            const int len = (int)min((int64_t)window, s1 - w0);
            int n = 0;   // uniform
            for (int e0 = 0; e0 < len; e0 += 64 * KI) {
                int key[KI];
#pragma unroll
                for (int u = 0; u < KI; ++u) {
                    const int e = e0 + 64 * u + l;
                    const int v = idx[(w0 + (e < len ? e : len - 1)) * N + k];
                    key[u] = e < len ? v : -1;
                }
#pragma unroll
                for (int u = 0; u < KI; ++u) {
                    const uint64_t m = __ballot(key[u] == i);
                    if (m) {   // uniform
                        if (key[u] == i) list[n + __popcll(m & ((1ull << l) - 1ull))] = (uint16_t)(e0 + 64 * u + l);
                        n += (int)__popcll(m);
                    }
                }
            }
            // this wavefront's LDS stores complete before its own reads
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int q0 = 0; q0 < n; q0 += 64) {
                ef4 acc = {0.f, 0.f, 0.f, 0.f};
                int nb = min(64, n - q0);
                const int64_t b = w0 + list[q0 + (l < nb ? l : nb - 1)];
                float rl = resid[b] * sc;
                OT off[NM - 1];   // this lane's entry: byte offsets of its slices of cores k+1, ..., k-1
                bool okl = l < nb;
                int ikk[NM - 1];
                int kk = k0;
#pragma unroll
                for (int q = 0; q < NM - 1; ++q) {
                    if (q >= N - 1) break;
                    ikk[q] = idx[b * N + kk];
                    kk = ring_next(kk, N);
                }
                kk = k0;
#pragma unroll
                for (int q = 0; q < NM - 1; ++q) {
                    if (q >= N - 1) break;
                    okl = okl && ikk[q] >= 0 && ikk[q] < d.I[kk];
                    off[q] = (OT)(uint32_t)ikk[q] * (OT)(4 * d.R[kk] * d.R[ring_next(kk, N)]);
                    kk = ring_next(kk, N);
                }
                const uint64_t okm = __ballot(okl);
                const int nv = (int)__popcll(okm);
                if (nv < nb) {   // uniform, rare: close the gaps the invalid entries leave
                    if (nv == 0) continue;
                    if (okl) list[q0 + __popcll(okm & ((1ull << l) - 1ull))] = (uint16_t)l;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    const int src = list[q0 + (l < nv ? l : nv - 1)];
                    rl = __shfl(rl, src, 64);
#pragma unroll
                    for (int q = 0; q < NM - 1; ++q)
                        if (q < N - 1) off[q] = (OT)__shfl(off[q], src, 64);
                    nb = nv;
                }
                // U packs: every pack's loads, then every pack's products;
                // TAIL: lanes past the batch compute on its last entry, masked
                auto round = [&](int at, auto tail) {
                    constexpr bool TAIL = decltype(tail)::value;
                    ef4 v[U][NM - 1];
                    float r[U];
                    uint32_t on[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int a0 = at + u * P + L.p, src = TAIL && a0 >= nb ? nb - 1 : a0;
                        on[u] = !TAIL || a0 < nb ? ~0u : 0u;
                        r[u] = __shfl(rl, src, 64);
                        int kc = k0;
#pragma unroll
                        for (int q = 0; q < NM - 1; ++q) {
                            if (q >= N - 1) break;
                            v[u][q] = sl.load(cores.p[kc], (OT)__shfl(off[q], src, 64), q);
                            kc = ring_next(kc, N);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        ef4 T = sl.template mask<TAIL>(v[u][0] * r[u], 0, on[u]);
                        int kc = k0;
#pragma unroll
                        for (int q = 1; q < NM - 1; ++q) {
                            if (q >= N - 1) break;
                            kc = ring_next(kc, N);
                            const ef4 a = sl.template mask<TAIL>(v[u][q], q, on[u]);
                            if (q + 1 < N - 1)
                                T = chain_mask(chain_mul(a, T, ef4{0.f, 0.f, 0.f, 0.f}), L, in0,
                                               d.R[ring_next(kc, N)]);
                            else
                                acc = chain_mul(a, T, acc);
                        }
                        if (N == 2) acc += T;
                    }
                };
                int at = 0;
#pragma unroll 1
                for (; at + U * P <= nb; at += U * P) round(at, std::false_type{});
                if (at < nb) round(at, std::true_type{});
#pragma unroll
                for (int j = 0; j < 4; ++j) tot[j] += (double)acc[j];
            }
        }
        // the packed blocks, then the wavefronts, in a fixed order
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (RB == 4) tot[j] += __shfl_xor(tot[j], 20, 64);
            if constexpr (RB <= 8) tot[j] += __shfl_xor(tot[j], 40, 64);
        }
        const int Rk = d.R[k], RR = Rk * d.R[k0];
        __syncthreads();   // every list has been read
        float* wsum = reinterpret_cast<float*>(smem_raw);   // [wavefronts][RB * RB]
        if (L.on[0] && L.p == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) wsum[w * (RB * RB) + L.col * RB + L.row[j]] = (float)tot[j];
        }
        __syncthreads();
        float* out = static_cast<float*>(grads.p[k]) + ((int64_t)part * d.I[k] + i) * RR;
        for (int e = tid; e < RR; e += blockDim.x) {
            const float* p = wsum + (e / Rk) * RB + e % Rk;
            double sum = 0.0;
            for (int v = 0; v < W; ++v) sum += (double)p[v * (RB * RB)];
            out[e] = (float)sum;
        }
        __syncthreads();   // the partial tiles have been read
    }
}

// Entry o of core k's gradient from its partial sums at ``g`` (mode k's), in part
// order.
__device__ __forceinline__ double entry_part_sum(const float* __restrict__ g, int64_t o, int parts, int64_t len) {
    double s = (double)g[o];
#pragma unroll 8
    for (int p = 1; p < parts; ++p) s += (double)g[o + p * len];
    return s;
}

// Element e of all cores, core after core: its core, its place there, the core's
// length.
__device__ __forceinline__ int entry_core_of(const tr_desc& d, int64_t e, int64_t* o, int64_t* len) {
    int k = 0;
    for (;; ++k) {
        *len = (int64_t)d.I[k] * d.R[k] * d.R[ring_next(k, d.N)];
        if (e < *len) break;
        e -= *len;
    }
    *o = e;
    return k;
}

// The gradients of the modes of several parts.
__global__ __launch_bounds__(256) void k_entry_bwd_sum(tr_desc d, const float* __restrict__ gpart, EntGroups gr,
                                                       int64_t slice_len, MutPtrs grads) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= slice_len) return;
    int64_t o, len;
    const int k = entry_core_of(d, e, &o, &len);
    if (gr.parts[k] > 1) static_cast<float*>(grads.p[k])[o] = (float)entry_part_sum(gpart + gr.at[k], o, gr.parts[k], len);
}

// Split of the batch.  A slice's workgroup gets more wavefronts until one's share
// is kBwdShare entries, unless there are so many slices that the wavefronts' fixed
// cost is what counts (kBwdSplit of them in all): a wavefront walks its hits in a
// chain of dependent loads, some 0.4 us an entry, so the share bounds it however
// the entries fall on the slices.  Modes of so few indices that a wavefront expects
// more than kBwdRounds rounds of hits, and batches past kBwdFar entries a wavefront,
// are split over several workgroups per slice, at most kBwdParts and kBwdPartBytes
// of partial gradients.
//
// Backward of uniform batches in us, one workgroup a slice with its wavefronts by
// the number of slices alone, against this split: sizes 2049, 5, 6, ranks 4/8/4, B
// 65536: 1946, 110; 14456, 826, 580, 9, 2, ranks 3/2/2/7/8, B 7975: 1445, 118; 2 and
// 145, ranks 16/6, B 15486: 100, 24; 1 and 1, ranks 16/12, B 65536: 685, 25; 10^6,
// ranks 7, B 8192: 96, 38; 16^4, ranks 11, B 32768: 227, 77.  Half of the batch on one
// index of every mode, 301 x 250 x 127, ranks 10/9/7, B 16384: 1136, 633 (uniform: 31).
// kBwdRounds 32: 132, 141, 34, 34, 60, 131; 8: 107, 109, 19, 27, 56, 82, but 60^4,
// ranks 10, B 16384: 50 instead of 41.  kBwdSplit 4 times as large: 150 and 162 for the
// first two.
constexpr int kBwdShare = 2048, kBwdRounds = 16, kBwdFar = 8192, kBwdParts = 512;
constexpr int64_t kBwdSplit = 1 << 15;
constexpr int64_t kBwdPartBytes = (int64_t)8 << 20;   // a mode

struct EntryPlan {
    int fwd_blocks, fwd_iters, rb, nm, waves, window;
    bool vec, big;   // big: a core of 4 GiB or more
    int64_t slice_len;
    EntGroups gr;
    int64_t part_len;                    // floats of the partial gradients
    size_t part_off, gpart_off, total;
};

static EntryPlan entry_plan(const tr_desc& d, int B) {
    EntryPlan P{};
    const Shape sh = shape_of(d);
    P.rb = sh.maxR <= 4 ? 4 : (sh.maxR <= 8 ? 8 : 16);
    for (int k = 0; k < d.N; ++k)
        P.big = P.big || (int64_t)d.I[k] * d.R[k] * d.R[ring_next(k, d.N)] >= ((int64_t)1 << 30);
    P.nm = P.big ? kMaxOrder : (d.N <= 3 ? 3 : (d.N <= 5 ? 5 : kMaxOrder));
    // one round per wavefront up to a full chip (four wavefronts per SIMD)
    const int64_t per = (kEntBlock / 64) * (16 / P.rb) * ent_packs(P.nm), fb = ((int64_t)B + per - 1) / per;
    P.fwd_iters = (int)std::min<int64_t>(16, (fb + 1023) / 1024);
    P.fwd_blocks = (int)((fb + P.fwd_iters - 1) / P.fwd_iters);
    P.vec = true;
    for (int k = 0; k < d.N; ++k) {
        const int64_t len = (int64_t)d.I[k] * d.R[k] * d.R[ring_next(k, d.N)];
        P.slice_len += len;
        P.gr.base[k + 1] = P.gr.base[k] + d.I[k];
        P.vec = P.vec && d.R[k] % 4 == 0;
    }
    // at most four wavefronts per SIMD over all slices, at least 64 entries of
    // scan each
    P.waves = 1;
    while (P.waves < bwd_waves(P.nm) && 2 * P.gr.base[d.N] * P.waves <= 4096 && (int64_t)64 * P.waves < B) P.waves *= 2;
    const int64_t slices = P.gr.base[d.N];
    while (P.waves < bwd_waves(P.nm) && (int64_t)kBwdShare * P.waves < B && 2 * slices * P.waves <= kBwdSplit) P.waves *= 2;
    for (int k = 0; k < d.N; ++k) {
        const int64_t len = (int64_t)d.I[k] * d.R[k] * d.R[ring_next(k, d.N)];
        const int64_t round = (16 / P.rb) * ent_packs(P.nm);   // entries of one
        const int64_t hits = std::min<int64_t>(d.I[k] * round * kBwdRounds, kBwdFar);
        const int64_t parts = std::min(std::min<int64_t>((B + hits * P.waves - 1) / (hits * P.waves), kBwdParts),
                                       kBwdPartBytes / (len * 4));
        P.gr.parts[k] = (int)std::max<int64_t>(1, parts);
        P.gr.base[k + 1] = P.gr.base[k] + (int64_t)d.I[k] * P.gr.parts[k];
        P.gr.at[k] = P.part_len;
        if (P.gr.parts[k] > 1) P.part_len += len * P.gr.parts[k];
    }
    const int64_t share = (((int64_t)B + P.waves - 1) / P.waves + 63) & ~(int64_t)63;
    P.window = (int)std::max<int64_t>(kBwdWindowMin, std::min<int64_t>(kBwdWindow, share));
    P.part_off = 0;
    P.gpart_off = align_up((size_t)std::max<int64_t>(P.fwd_blocks, std::min<int64_t>(fb, 1024)) * 8);
    P.total = P.gpart_off + align_up((size_t)P.part_len * 4);
    return P;
}

// Largest ``bytes`` of a batch of at most B entries, so that the workspace of the
// largest batch serves smaller ones: the forward's blocks fall where its wavefronts
// take one round more, a mode's parts where a workgroup gets more wavefronts (at 64
// or kBwdShare entries for each); between those sizes neither falls.  211, 1, 290,
// 45, ranks 13/1/3/15: 78592 bytes for B 7472, 5376 for B 9230.
template <typename F>
static size_t entry_size_upto(int B, F&& bytes) {
    size_t most = bytes(B);
    for (int w = 1; w <= 8; w *= 2) {
        if (64 * w < B) most = std::max(most, bytes(64 * w));
        if (kBwdShare * w < B) most = std::max(most, bytes(kBwdShare * w));
    }
    return most;
}

// 16-byte slice loads: every rank a multiple of 4 (so every slice is whole
// pieces) and every core 16-byte aligned.
static bool entry_vec(const tr_desc& d, const EntryPlan& P, const Ptrs& cp) {
    bool v = P.vec;
    for (int k = 0; k < d.N; ++k) v = v && (reinterpret_cast<uintptr_t>(cp.p[k]) & 15) == 0;
    return v;
}

// ------------------------------------------------------------ completion --
//
// Tensor completion with a ridge term on the sampled-entry loss: per step,
// B observed entries drawn uniformly with replacement (position
// floor(r |Omega| / 2^64), r from Philox counter (t, b, 0, TR_STREAM_ENTRY)),
// the forward and backward above, then G_k <- rule(G_k, p) with
// p = -(dL/dG_k + lambda G_k) for every core, or for core n = the step's
// mode only.

template <typename TX>
__global__ __launch_bounds__(256) void k_completion_draw(tr_desc d, const uint64_t* __restrict__ t_dev,
                                                         uint64_t seed, const int32_t* __restrict__ obs_idx,
                                                         const TX* __restrict__ obs_x, int64_t n_obs, int B,
                                                         int32_t* __restrict__ bidx, TX* __restrict__ bx) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const uint64_t t = *t_dev;
    const int64_t j = (int64_t)mulhi64(draw_word(seed, t, (uint64_t)b, 0, TR_STREAM_ENTRY), (uint64_t)n_obs);
    for (int k = 0; k < d.N; ++k) bidx[(int64_t)b * d.N + k] = obs_idx[j * d.N + k];
    bx[b] = obs_x[j];
}

// loss = 1/(2B) sum r^2 (the forward's block partials, in block order) +
// lambda/2 sum_k ||G_k||^2 (each strided per thread, then the block tree).
__global__ __launch_bounds__(1024) void k_completion_loss(tr_desc d, const double* __restrict__ part, int nb, int B,
                                                          Ptrs cores, double lam, double* __restrict__ loss) {
    __shared__ double red[16];
    double s = 0.0;
    if (lam != 0.0)
        for (int k = 0; k < d.N; ++k) {
            const float* G = static_cast<const float*>(cores.p[k]);
            const int64_t len = (int64_t)d.I[k] * d.R[k] * d.R[ring_next(k, d.N)];
#pragma unroll 8
            for (int64_t e = threadIdx.x; e < len; e += blockDim.x) s += (double)G[e] * (double)G[e];
        }
    const double ridge = block_sum(s, red);
    double data = 0.0;
    for (int q = threadIdx.x; q < nb; q += blockDim.x) data += part[q];
    data = block_sum(data, red);
    if (threadIdx.x == 0) *loss = data / (2.0 * (double)B) + 0.5 * lam * ridge;
}

// The update; its last block advances the step counter.
__global__ __launch_bounds__(256) void k_completion_update(tr_desc d, const uint64_t* __restrict__ t_dev,
                                                           uint64_t seed, int block, MutPtrs cores, MutPtrs accum,
                                                           const float* __restrict__ grads, EntGroups gr, int64_t slice_len,
                                                           double lam, tr_step rule, int32_t* status, StepBump step) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool reads_t = block || rule.kind == 2;
    if (e < slice_len) {
        const uint64_t t = reads_t ? *t_dev : 0;
        int64_t o, len;
        const int k = entry_core_of(d, e, &o, &len);
        if (!block || k == pick_mode(seed, t, d.N)) {
            float* G = static_cast<float*>(cores.p[k]);
            float* A = static_cast<float*>(accum.p[k]);
            const double p = -(entry_part_sum(grads + gr.at[k], o, gr.parts[k], len) + lam * (double)G[o]);
            apply_rule(G, A, o, p, rule, t, status);
        }
    }
    bump_if_last(step, reads_t);
}

// F::run<RB, VEC, NM, OT>(args...) for the plan's kernel variant.
template <typename F, int RB, bool VEC, typename... A>
static void entry_dispatch_nm(const EntryPlan& P, A... a) {
    // (cores of 4 GiB and more are rare enough to take the widest order's form)
    if (P.big) F::template run<RB, VEC, kMaxOrder, uint64_t>(a...);
    else if (P.nm == 3) F::template run<RB, VEC, 3, uint32_t>(a...);
    else if (P.nm == 5) F::template run<RB, VEC, 5, uint32_t>(a...);
    else F::template run<RB, VEC, kMaxOrder, uint32_t>(a...);
}
template <typename F, typename... A>
static void entry_dispatch(const EntryPlan& P, bool vec, A... a) {
    if (P.rb == 4) vec ? entry_dispatch_nm<F, 4, true>(P, a...) : entry_dispatch_nm<F, 4, false>(P, a...);
    else if (P.rb == 8) vec ? entry_dispatch_nm<F, 8, true>(P, a...) : entry_dispatch_nm<F, 8, false>(P, a...);
    else vec ? entry_dispatch_nm<F, 16, true>(P, a...) : entry_dispatch_nm<F, 16, false>(P, a...);
}

template <typename TX>
struct FwdLaunch {
    template <int RB, bool VEC, int NM, typename OT>
    static void run(const tr_desc* d, const EntryPlan* P, Ptrs cp, const int32_t* idx, const TX* x, int B,
                    float* resid, double* part, hipStream_t st) {
        hipLaunchKernelGGL((k_entry_fwd<TX, RB, VEC, NM, OT>), dim3(P->fwd_blocks), dim3(kEntBlock), 0, st, *d, cp,
                           idx, x, B, P->fwd_iters, resid, part);
    }
};

template <typename TX>
static void launch_entry_fwd(const tr_desc& d, const EntryPlan& P, Ptrs cp, const int32_t* idx, const TX* x, int B,
                             float* resid, double* part, hipStream_t st) {
    entry_dispatch<FwdLaunch<TX>>(P, entry_vec(d, P, cp), &d, &P, cp, idx, x, B, resid, part, st);
}

struct BwdLaunch {
    template <int RB, bool VEC, int NM, typename OT>
    static void run(const tr_desc* d, const EntryPlan* P, Ptrs cp, const int32_t* idx, const float* resid, int B,
                    float scale, const double* scale_dev, ModeSrc only, int block, MutPtrs grads, hipError_t* e,
                    hipStream_t st) {
        const size_t shm = (size_t)P->waves * P->window * 2;
        if (!allow_lds(reinterpret_cast<const void*>(&k_entry_bwd<RB, VEC, NM, OT>), shm)) {
            *e = hipErrorInvalidValue;
            return;
        }
        hipLaunchKernelGGL((k_entry_bwd<RB, VEC, NM, OT>), dim3((unsigned)std::min(P->gr.base[d->N], kBwdGrid)),
                           dim3(64 * P->waves), shm, st, *d, cp, idx, resid, B, scale, scale_dev, P->gr,
                           P->window, only, block, grads);
        *e = hipGetLastError();
    }
};

// ``block`` nonzero: only the core of ``only``'s mode.  grads: of a mode of several
// parts its partial sums.
static hipError_t launch_entry_bwd(const tr_desc& d, const EntryPlan& P, Ptrs cp, const int32_t* idx,
                                   const float* resid, int B, float scale, const double* scale_dev, ModeSrc only,
                                   int block, MutPtrs grads, hipStream_t st) {
    hipError_t e = hipSuccess;
    entry_dispatch<BwdLaunch>(P, entry_vec(d, P, cp), &d, &P, cp, idx, resid, B, scale, scale_dev, only, block, grads,
                              &e, st);
    return e;
}

struct CompletionWs {
    EntryPlan P;
    size_t bidx, bx, resid, grads, ctr, total;
};

static CompletionWs completion_layout(const tr_desc& d, int B) {
    CompletionWs L{};
    L.P = entry_plan(d, B);
    size_t o = align_up(L.P.gpart_off);   // the forward's part of the plan; the gradient parts are ``grads``
    L.bidx = o;
    o += align_up((size_t)B * d.N * 4);
    L.bx = o;
    o += align_up((size_t)B * 4);
    L.resid = o;
    o += align_up((size_t)B * 4);
    L.grads = o;
    int64_t len = 0;   // every mode's partial sums, or its gradient
    for (int k = 0; k < d.N; ++k) {
        L.P.gr.at[k] = len;
        len += (int64_t)d.I[k] * d.R[k] * d.R[ring_next(k, d.N)] * L.P.gr.parts[k];
    }
    o += align_up((size_t)len * 4);
    L.ctr = o;
    o += align_up(4);
    L.total = o;
    return L;
}

}  // namespace trk

using namespace trk;

extern "C" {

size_t tr_entry_workspace_size(const tr_desc* d, int32_t B) {
    if (validate_desc(d) != TR_OK || B < 1) return 0;
    return entry_size_upto(B, [&](int b) { return entry_plan(*d, b).total; });
}

static tr_status entry_checks(const tr_desc* d, const void* const* cores, const int32_t* idx, int32_t B) {
    tr_status s = validate_desc(d);
    if (s != TR_OK) return s;
    if (d->core_dtype != TR_F32) return TR_E_DTYPE;
    if (!cores || !idx) return TR_E_ARG;
    for (int k = 0; k < d->N; ++k)
        if (!cores[k]) return TR_E_ARG;
    if (B < 1 || B > (1 << 26)) return TR_E_SHAPE;
    return TR_OK;
}

tr_status tr_entry_fwd(const tr_desc* d, const void* const* cores, const int32_t* idx, const void* x, int32_t B,
                       float* resid, double* loss, void* ws, size_t ws_bytes, tr_stream_t stream) {
    tr_status s = entry_checks(d, cores, idx, B);
    if (s != TR_OK) return s;
    if (!x || !resid) return TR_E_ARG;
    const EntryPlan P = entry_plan(*d, B);
    if (!ws || ws_bytes < P.total) return TR_E_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    Ptrs cp{};
    for (int k = 0; k < d->N; ++k) cp.p[k] = cores[k];
    double* part = reinterpret_cast<double*>(static_cast<char*>(ws) + P.part_off);
    switch (d->x_dtype) {
        case TR_F32:
            launch_entry_fwd(*d, P, cp, idx, static_cast<const float*>(x), B, resid, part, st);
            break;
        case TR_F16:
            launch_entry_fwd(*d, P, cp, idx, static_cast<const __half*>(x), B, resid, part, st);
            break;
        default:
            return TR_E_DTYPE;
    }
    if (hipGetLastError() != hipSuccess) return TR_E_HIP;
    if (loss) {
        hipLaunchKernelGGL(k_entry_loss, dim3(1), dim3(256), 0, st, part, P.fwd_blocks, B, loss);
        if (hipGetLastError() != hipSuccess) return TR_E_HIP;
    }
    return TR_OK;
}

tr_status tr_entry_bwd(const tr_desc* d, const void* const* cores, const int32_t* idx, const float* resid, int32_t B,
                       double scale, const double* scale_dev, void* const* grads, void* ws, size_t ws_bytes,
                       tr_stream_t stream) {
    tr_status s = entry_checks(d, cores, idx, B);
    if (s != TR_OK) return s;
    if (!resid || !grads) return TR_E_ARG;
    for (int k = 0; k < d->N; ++k)
        if (!grads[k]) return TR_E_ARG;
    const EntryPlan P = entry_plan(*d, B);
    if (!ws || ws_bytes < P.total) return TR_E_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    Ptrs cp{};
    MutPtrs gp{};
    float* gpart = reinterpret_cast<float*>(static_cast<char*>(ws) + P.gpart_off);
    MutPtrs to{};   // where the slices go: grads, or the parts
    for (int k = 0; k < d->N; ++k) {
        cp.p[k] = cores[k];
        gp.p[k] = grads[k];
        to.p[k] = P.gr.parts[k] > 1 ? static_cast<void*>(gpart + P.gr.at[k]) : grads[k];
    }
    hipError_t e = launch_entry_bwd(*d, P, cp, idx, resid, B, (float)scale, scale_dev, ModeSrc{}, 0, to, st);
    if (e == hipSuccess && P.part_len > 0) {
        hipLaunchKernelGGL(k_entry_bwd_sum, dim3((unsigned)((P.slice_len + 255) / 256)), dim3(256), 0, st, *d, gpart,
                           P.gr, P.slice_len, gp);
        e = hipGetLastError();
    }
    return e == hipSuccess ? TR_OK : TR_E_HIP;
}

static tr_status completion_checks(const tr_desc* d, const tr_completion_config* c) {
    tr_status s = validate_desc(d);
    if (s != TR_OK) return s;
    if (!c) return TR_E_ARG;
    if (d->core_dtype != TR_F32) return TR_E_DTYPE;
    if (d->x_dtype != TR_F32 && d->x_dtype != TR_F16) return TR_E_DTYPE;
    if (c->B < 1 || c->B > (1 << 26)) return TR_E_SHAPE;
    if (!(c->lambda >= 0.0)) return TR_E_ARG;
    if (c->rule.kind < 0 || c->rule.kind > 2) return TR_E_ARG;
    if (c->rule.kind == 2 && !(c->rule.tau > 0.0)) return TR_E_ARG;
    return TR_OK;
}

size_t tr_completion_workspace_size(const tr_desc* d, const tr_completion_config* c) {
    if (completion_checks(d, c) != TR_OK) return 0;
    return entry_size_upto(c->B, [&](int b) { return completion_layout(*d, b).total; });
}

tr_status tr_completion_run(const tr_desc* d, void* const* cores, void* const* accum, const int32_t* obs_idx,
                            const void* obs_x, int64_t n_obs, const tr_completion_config* c, uint64_t* t_dev,
                            int32_t steps, double* loss_out, int32_t* dev_status, void* ws, size_t ws_bytes,
                            tr_stream_t stream) {
    tr_status s = completion_checks(d, c);
    if (s != TR_OK) return s;
    if (!cores || !obs_idx || !obs_x || !t_dev || n_obs < 1 || steps < 0) return TR_E_ARG;
    for (int k = 0; k < d->N; ++k) {
        if (!cores[k]) return TR_E_ARG;
        if (c->rule.kind == 1 && (!accum || !accum[k])) return TR_E_ARG;
    }
    const CompletionWs L = completion_layout(*d, c->B);
    if (!ws || ws_bytes < L.total) return TR_E_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return TR_E_ALIGN;
    if (steps == 0) return TR_OK;
    hipStream_t st = (hipStream_t)stream;
    char* w = static_cast<char*>(ws);
    double* part = reinterpret_cast<double*>(w + L.P.part_off);
    int32_t* bidx = reinterpret_cast<int32_t*>(w + L.bidx);
    float* resid = reinterpret_cast<float*>(w + L.resid);
    float* grads = reinterpret_cast<float*>(w + L.grads);
    unsigned* ctr = reinterpret_cast<unsigned*>(w + L.ctr);
    Ptrs cp{};
    MutPtrs mc{}, ac{}, gp{};
    for (int k = 0; k < d->N; ++k) {
        cp.p[k] = cores[k];
        mc.p[k] = cores[k];
        ac.p[k] = accum ? accum[k] : nullptr;
        gp.p[k] = grads + L.P.gr.at[k];
    }
    const int B = c->B;
    const dim3 gd((unsigned)((B + 255) / 256));
    const dim3 gu((unsigned)((L.P.slice_len + 255) / 256));
    if (launch_zero_u32(ctr, 1, st) != hipSuccess) return TR_E_HIP;
    const ModeSrc only{t_dev, 0, -1, c->seed, nullptr, nullptr};
    for (int it = 0; it < steps; ++it) {
        if (d->x_dtype == TR_F32) {
            float* bx = reinterpret_cast<float*>(w + L.bx);
            hipLaunchKernelGGL(k_completion_draw<float>, gd, dim3(256), 0, st, *d, t_dev, c->seed, obs_idx,
                               static_cast<const float*>(obs_x), n_obs, B, bidx, bx);
            launch_entry_fwd(*d, L.P, cp, bidx, static_cast<const float*>(bx), B, resid, part, st);
        } else {
            __half* bx = reinterpret_cast<__half*>(w + L.bx);
            hipLaunchKernelGGL(k_completion_draw<__half>, gd, dim3(256), 0, st, *d, t_dev, c->seed, obs_idx,
                               static_cast<const __half*>(obs_x), n_obs, B, bidx, bx);
            launch_entry_fwd(*d, L.P, cp, bidx, static_cast<const __half*>(bx), B, resid, part, st);
        }
        if (loss_out)
            hipLaunchKernelGGL(k_completion_loss, dim3(1), dim3(1024), 0, st, *d, part, L.P.fwd_blocks, B, cp,
                               c->lambda, loss_out + it);
        if (launch_entry_bwd(*d, L.P, cp, bidx, resid, B, 1.0f, nullptr, only, (int)c->block, gp, st) != hipSuccess)
            return TR_E_HIP;
        hipLaunchKernelGGL(k_completion_update, gu, dim3(256), 0, st, *d, t_dev, c->seed, (int)c->block, mc, ac,
                           grads, L.P.gr, L.P.slice_len, c->lambda, c->rule, dev_status, StepBump{t_dev, ctr});
        if (hipGetLastError() != hipSuccess) return TR_E_HIP;
    }
    return TR_OK;
}

}  // extern "C"
