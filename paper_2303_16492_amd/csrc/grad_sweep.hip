// a5-a7 of a scaled step on one stream: the gradient's 16-byte forms and the inverse
// of the Gram in one launch, since neither needs the other's result.  Workgroup 0
// inverts (sweep.hpp); the gradient's blocks (grad_wide.hpp, mixed_wide.hpp) start
// at workgroup 8, so that each stays on its XCD.
//
// Bound: the inverse's chain of pivots (22 us at R_n R_{n+1} = 100), the gradient's
// 16 us beside it.  Every workgroup reserves the LDS of a CU: the gradient's one
// block a CU is the form's own layout, and no other work stretches the chain on the
// inverse's SIMDs.  A kernel has the registers of the inverse, one wavefront a SIMD.
// 400^3, ranks 10, m 4096, FP32: 22.9 us for both (22.6 for the inverse alone, 15.8
// for the gradient); a captured step 52.5 us, 66.3 with one launch after the other,
// 53.3 with the two on two streams.  The forms not served here take little beside
// what a second stream's events cost: FP16, 30 x 20 x 60 x 300, ranks 3, m 1600, one
// launch after the other 37.8 us a captured step.
#include "grad_wide.hpp"
#include "mixed_wide.hpp"
#include "sweep.hpp"

namespace trk {

constexpr unsigned kSweepSlots = 8;   // workgroups before the gradient's: the inverse and seven that end at once

struct SweepArgs {
    ModeSrc ms;
    const double* gram;
    Damp damp;
    double* hm;
    int* flag;
    int32_t* status;
};

template <int NT>
__device__ __forceinline__ void sweep_slot(const tr_desc& d, const SweepArgs& a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if (blockIdx.x == 0)
        sweep_block<NT>(d, a.ms, a.gram, a.damp, 0.0, a.hm, a.flag, a.status, *reinterpret_cast<SweepShared*>(smem_raw));
}

template <typename TX, int CT>
__global__ __launch_bounds__(256) void k_sweep_grad_f32w(tr_desc d, SweepArgs sa, ModeSrc ms, Ptrs cores, XSrc xsrc,
                                                         const int32_t* __restrict__ idx,
                                                         const float* __restrict__ S, const double* __restrict__ pF,
                                                         int m, int groups, int row_tiles, float* __restrict__ gp,
                                                         double* __restrict__ lp, int maxIRR, int rr_fixed,
                                                         WideModes tab) {
    if (blockIdx.x < kSweepSlots)
        sweep_slot<CT>(d, sa);
    else
        grad_f32w_block<TX, CT>((int)(blockIdx.x - kSweepSlots), d, ms, cores, xsrc, idx, S, pF, m, groups, row_tiles,
                                gp, lp, maxIRR, rr_fixed, tab);
}

template <typename T16, typename TX, int CT>
__global__ __launch_bounds__(256) void k_sweep_grad_mixed_w(tr_desc d, SweepArgs sa, ModeSrc ms, Ptrs cores,
                                                            XSrc xsrc, const int32_t* __restrict__ idx,
                                                            const float* __restrict__ S,
                                                            const double* __restrict__ pF, int m, int groups,
                                                            int row_tiles, float* __restrict__ gp,
                                                            double* __restrict__ lp, int maxIRR, int rr_fixed,
                                                            WideModes tab) {
    if (blockIdx.x < kSweepSlots)
        sweep_slot<CT>(d, sa);
    else
        grad_mixed_w_block<T16, TX, CT>((int)(blockIdx.x - kSweepSlots), d, ms, cores, xsrc, idx, S, pF, m, groups,
                                        row_tiles, gp, lp, maxIRR, rr_fixed, tab);
}

template <typename F>
static hipError_t launch_both(F kern, size_t shm, dim3 grid, hipStream_t st, const tr_desc& d, const SweepArgs& sa,
                              ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx, const float* S, const double* pF,
                              int m, const GradWs& L, float* gp, double* lp, size_t xelem) {
    // all of a CU's LDS but 1 KB (the gradient's own sums are static)
    constexpr size_t kReserve = 159 * 1024;
    static_assert(sizeof(SweepShared) <= kReserve, "the inverse lives in the dynamic LDS");
    if (shm > kReserve || !allow_lds(reinterpret_cast<const void*>(kern), kReserve)) return hipErrorNotSupported;
    const Shape sh = shape_of(d);
    hipLaunchKernelGGL(kern, grid, dim3(256), kReserve, st, d, sa, ms, cores, xs, idx, S, pF, m, L.groups, L.row_tiles,
                       gp, lp, sh.maxI * sh.maxRR, wide_rr_fixed(d), wide_modes(d, xs, m, xelem));
    return hipGetLastError();
}

// hipErrorNotSupported, and nothing launched, where the two go one after the other:
// FP64, shapes that the 16-byte forms do not take, and grids of more blocks than CUs
// (a block that waits for a CU would start after the inverse's or the first blocks').
hipError_t launch_sweep_grad(const tr_desc& d, ModeSrc ms_shape, const double* gram, Damp damping, const UpdWs& U,
                             void* upd_ws, int32_t* status, ModeSrc ms, Ptrs cores, XSrc xs, const int32_t* idx,
                             const void* S, const double* pF, int m, int prec, void* grad_ws, const GradWs& L,
                             hipStream_t st) {
    constexpr unsigned kCus = 256;
    if (d.core_dtype != TR_F32 || (d.x_dtype != TR_F32 && d.x_dtype != TR_F16)) return hipErrorNotSupported;
    const Shape sh = shape_of(d);
    char *w = static_cast<char*>(grad_ws), *u = static_cast<char*>(upd_ws);
    float* gp = reinterpret_cast<float*>(w + L.gpart_off);
    double* lp = reinterpret_cast<double*>(w + L.lpart_off);
    const float* Sf = static_cast<const float*>(S);
    const unsigned blocks = kSweepSlots + xcd_grid(L.row_tiles, L.groups);
    if (!wide_applies(d, cores, Sf, gp, m, L.groups, sh.maxRR, kWideTF) || blocks > kCus) return hipErrorNotSupported;
    const SweepArgs sa{ms_shape, gram, damping, reinterpret_cast<double*>(u + U.L_off),
                       reinterpret_cast<int*>(u + U.flag_off), status};
    const bool xf = d.x_dtype == TR_F32;
    const size_t xelem = xf ? 4 : 2;
#define TRK_BOTH(KERN, SHM) \
    launch_both(KERN, SHM, dim3(blocks), st, d, sa, ms, cores, xs, idx, Sf, pF, m, L, gp, lp, xelem)
#define TRK_BOTH_CT(CT)                                                                                             \
    case CT:                                                                                                        \
        if (prec == TR_PREC_BF16)                                                                                   \
            return xf ? TRK_BOTH((&k_sweep_grad_mixed_w<__bf16, float, CT>), MixWideCfg<CT>::lds())                 \
                      : TRK_BOTH((&k_sweep_grad_mixed_w<__bf16, __half, CT>), MixWideCfg<CT>::lds());               \
        if (prec == TR_PREC_F16)                                                                                    \
            return xf ? TRK_BOTH((&k_sweep_grad_mixed_w<_Float16, float, CT>), MixWideCfg<CT>::lds())               \
                      : TRK_BOTH((&k_sweep_grad_mixed_w<_Float16, __half, CT>), MixWideCfg<CT>::lds());             \
        return xf ? TRK_BOTH((&k_sweep_grad_f32w<float, CT>), WideCfg<CT>::shm())                                   \
                  : TRK_BOTH((&k_sweep_grad_f32w<__half, CT>), WideCfg<CT>::shm())
    switch ((sh.maxRR + 15) / 16) {
        TRK_BOTH_CT(3);
        TRK_BOTH_CT(4);
        TRK_BOTH_CT(5);
        TRK_BOTH_CT(6);
        TRK_BOTH_CT(7);
        TRK_BOTH_CT(8);
        default: return hipErrorNotSupported;
    }
#undef TRK_BOTH_CT
#undef TRK_BOTH
}

}  // namespace trk
