// Integer-weight CDFs of one block: weights floor(p 2^40) + 1 and their
// inclusive prefix sums.
#pragma once
#include "internal.hpp"

namespace trk {

constexpr double kTwo40 = 1099511627776.0;

// Inclusive scan of a[0..len) (uint64) by one block, in place: each thread
// scans a contiguous segment, the segment sums are scanned across lanes with
// shuffles and across wavefronts through LDS, and each segment adds its
// offset.  Integer sums: the result does not depend on the grouping.
__device__ inline void block_scan_u64(uint64_t* a, int64_t len) {
    __shared__ uint64_t wtot[16];
    const int T = blockDim.x, lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (T + 63) >> 6;
    const int64_t per = (len + T - 1) / T;
    const int64_t b = threadIdx.x * per, e = min(len, b + per);
    uint64_t s = 0;
    for (int64_t i = b; i < e; ++i) {
        s += a[i];
        a[i] = s;
    }
    uint64_t incl = s;   // inclusive scan of the segment sums within the wavefront
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(incl, (unsigned)o, 64);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wtot[wid] = incl;
    __syncthreads();
    if (wid == 0) {   // exclusive scan of the wavefront totals
        const uint64_t v = lane < nw ? wtot[lane] : 0ull;
        uint64_t x = v;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const uint64_t y = __shfl_up(x, (unsigned)o, 64);
            if (lane >= o) x += y;
        }
        if (lane < nw) wtot[lane] = x - v;
    }
    __syncthreads();
    const uint64_t off = wtot[wid] + incl - s;
    for (int64_t i = b; i < e; ++i) a[i] += off;
    __syncthreads();
}

__device__ inline uint64_t quantize(double p) { return (uint64_t)floor(p * kTwo40) + 1ull; }

__device__ inline void write_uniform_weights(uint64_t* w, int64_t len) {
    const uint64_t wu = quantize(1.0 / (double)len);
    for (int64_t i = threadIdx.x; i < len; i += blockDim.x) w[i] = wu;
    __syncthreads();
}

// Weights staged in LDS when every core has at most this many rows (the
// launch then passes lds_rows = max I_k, else 0).
constexpr int kLdsRows = 8192;
constexpr int kLevLdsRows = 4096;

// w (Ik weights, in LDS or global memory) -> inclusive CDF in cdf; the
// step counter advances afterwards when ``bump`` is set (every thread of
// the block read it before the block's first barrier).
__device__ inline void finish_cdf(uint64_t* w, uint64_t* cdf, int Ik, uint64_t* bump) {
    block_scan_u64(w, Ik);
    if (w != cdf)
        for (int i = threadIdx.x; i < Ik; i += blockDim.x) cdf[i] = w[i];
    if (bump && threadIdx.x == 0) atomicAdd(reinterpret_cast<unsigned long long*>(bump), 1ull);
}

}  // namespace trk
