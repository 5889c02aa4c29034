// Products of FP32 core slices on the matrix cores (16 x 16 x 4) that never leave
// the registers.  With T = S_1 ... S_q the transposed product T^T sits in the
// result layout (entry j of a lane: row 4 (l / 16) + j, column l % 16), which is
// also the B operand of the next product T^T <- S^T T^T when K step j takes
// k = 4 (l / 16) + j, and the A operand of that step is S(4 (l / 16) + j, l % 16):
// four consecutive entries of a stored slice.
//
// Slices of ranks <= RB = 8 (4) are packed as 2 (4) diagonal blocks of one
// operand, one sample or entry each: block p of a lane is (l % 16) / RB.
#pragma once
#include "internal.hpp"

namespace trk {

typedef float chain4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float chain_and(float v, uint32_t m) { return __uint_as_float(__float_as_uint(v) & m); }

// A lane's place in an operand of 16 / RB diagonal RB x RB blocks: block p,
// column col inside it, and per entry j its row inside the block and whether
// that row lies in the same block (entries off the diagonal blocks are zero).
template <int RB>
struct ChainLane {
    int p, col, row[4];
    bool on[4];
    __device__ __forceinline__ ChainLane() {
        const int l = threadIdx.x & 63, lr = l & 15, lk = l >> 4;
        p = lr / RB;
        col = lr % RB;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 4 * lk + j;
            row[j] = r % RB;
            on[j] = r / RB == p;
        }
    }
};

// Byte offsets inside a slice of the four entries a lane loads, and their
// masks, for the slices of a chain of ``n`` cores from k0 (n <= NM): the first
// slice transposed, S(col, row), the others S(row, col).  Offsets are clamped
// into the slice; VEC: whole 16-byte pieces, every R_k a multiple of 4
// (only the first offset of the later slices is used).
template <int NM, bool VEC>
struct ChainSlots {
    uint32_t lo[NM][4], mk[NM][4];
    template <int RB>
    __device__ __forceinline__ ChainSlots(const tr_desc& d, int k0, int n, const ChainLane<RB>& L) {
        int k = k0;
#pragma unroll
        for (int q = 0; q < NM; ++q) {
            if (q >= n) break;
            const int Rk = d.R[k], Rk1 = d.R[ring_next(k, d.N)];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = q == 0 ? L.col : L.row[j], c = q == 0 ? L.row[j] : L.col;
                mk[q][j] = L.on[j] && r < Rk && c < Rk1 ? ~0u : 0u;
                const int rc = r < Rk ? r : (VEC && q > 0 ? 0 : Rk - 1), cc = c < Rk1 ? c : Rk1 - 1;
                lo[q][j] = (uint32_t)sizeof(float) * (uint32_t)(rc + Rk * cc);
            }
            k = ring_next(k, d.N);
        }
    }
    // the lane's entries of slice q of the chain, the slice at byte ``off`` of
    // its core (OT holds a byte offset into any core)
    template <typename OT>
    __device__ __forceinline__ chain4 load(const void* __restrict__ core, OT off, int q) const {
        const char* A = static_cast<const char*>(core);
        chain4 v;
        if constexpr (VEC) {
            if (q > 0) {
                const float4 w = *reinterpret_cast<const float4*>(A + (OT)(off + lo[q][0]));
                return chain4{w.x, w.y, w.z, w.w};
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const float*>(A + (OT)(off + lo[q][j]));
        return v;
    }
    // exact zeros outside the slice (an infinity or NaN of one packed slice
    // stays its own); ALSO: and where ``also`` is zero
    template <bool ALSO = false>
    __device__ __forceinline__ chain4 mask(chain4 v, int q, uint32_t also = ~0u) const {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = chain_and(v[j], ALSO ? mk[q][j] & also : mk[q][j]);
        return v;
    }
};

// acc + S^T T^T
__device__ __forceinline__ chain4 chain_mul(const chain4& a, const chain4& t, chain4 acc) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], t[j], acc, 0, 0, 0);
    return acc;
}

// A product's result with exact zeros outside its R0 x Rc block (in0: the
// lane's column is below R0, the rows of the chain's first slice).
template <int RB>
__device__ __forceinline__ chain4 chain_mask(chain4 v, const ChainLane<RB>& L, bool in0, int Rc) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = chain_and(v[j], in0 && L.on[j] && L.row[j] < Rc ? ~0u : 0u);
    return v;
}

}  // namespace trk
