// a8: the plain step (eq:update_brsgd or the AdaGrad remark) applied to a
// gradient already reduced, and the workspace of the scaled step.
#include "internal.hpp"

namespace trk {

template <typename TC>
__global__ __launch_bounds__(256) void k_plain_update(tr_desc d, ModeSrc ms, const TC* __restrict__ g,
                                                      MutPtrs cores, MutPtrs accum, tr_step rule,
                                                      int32_t* status) {
    uint64_t t;
    int n;
    resolve_mode(ms, d.N, &t, &n);
    const int64_t total = (int64_t)d.I[n] * d.R[n] * d.R[ring_next(n, d.N)];
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    TC* G = static_cast<TC*>(cores.p[n]);
    TC* A = static_cast<TC*>(accum.p[n]);
    apply_rule<TC>(G, A, e, -(double)g[e], rule, t, status);
}

UpdWs upd_ws_layout(const tr_desc& d) {
    UpdWs L{};
    const Shape sh = shape_of(d);
    L.L_off = 0;
    L.flag_off = align_up((size_t)sh.maxRR * sh.maxRR * 8);
    L.total = L.flag_off + 256;
    return L;
}

hipError_t launch_plain_update(const tr_desc& d, ModeSrc ms, const void* g, MutPtrs cores, MutPtrs accum,
                               tr_step rule, int32_t* status, hipStream_t st) {
    const Shape sh = shape_of(d);
    const dim3 grid((unsigned)(((int64_t)sh.maxI * sh.maxRR + 255) / 256));
    if (d.core_dtype == TR_F64)
        hipLaunchKernelGGL(k_plain_update<double>, grid, dim3(256), 0, st, d, ms, static_cast<const double*>(g),
                           cores, accum, rule, status);
    else
        hipLaunchKernelGGL(k_plain_update<float>, grid, dim3(256), 0, st, d, ms, static_cast<const float*>(g),
                           cores, accum, rule, status);
    return hipGetLastError();
}

}  // namespace trk
