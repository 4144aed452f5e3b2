// One L-BFGS update per fit, one wave each (lbfgs_device.hpp).
#include "lbfgs_device.hpp"

namespace pwa {
namespace {

__global__ __launch_bounds__(64) void lbfgs_kernel(const MultiFit *fits, const double *out, int64_t ostride,
                                                   LbfgsState *states, double c1, double ftol) {
    __shared__ double prod[64 * kLbfgsPer];
    const int f = blockIdx.x, n = 2 * fits[f].k;
    const double *o = out + (int64_t)f * ostride;
    const double ft = o[0];
    const LbVec gt = lb_load(o + 1, n, threadIdx.x);
    LbRegs r;
    lbfgs_load(r, states + f, n, false);
    lbfgs_advance(states + f, r, n, ft, gt, c1, ftol, false, 0.0, prod);
}

}  // namespace

hipError_t launch_lbfgs(const MultiFit *fits, const double *out, int64_t ostride, LbfgsState *states, int nfits, int m,
                        double c1, double ftol, hipStream_t stream) {
    if (m != kLbfgsHist) return hipErrorInvalidValue;
    hipLaunchKernelGGL(lbfgs_kernel, dim3(nfits), dim3(64), 0, stream, fits, out, ostride, states, c1, ftol);
    return hipGetLastError();
}

}  // namespace pwa
