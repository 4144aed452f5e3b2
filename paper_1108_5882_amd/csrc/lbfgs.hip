// One L-BFGS update per fit, one wave each (lbfgs_device.hpp).
#include "lbfgs_device.hpp"

namespace pwa {
namespace {

__global__ __launch_bounds__(64) void lbfgs_kernel(const MultiFit *fits, int k_all, const double *out, int64_t ostride,
                                                   LbfgsState *states, double c1, double ftol, int polar, double rmin) {
    __shared__ double prod[64 * kLbfgsPer];
    const int f = blockIdx.x;
    const double *o = out + (int64_t)f * ostride;
    lbfgs_advance(states + f, 2 * (fits ? fits[f].k : k_all), o[0], o + 1, c1, ftol, polar != 0, rmin, prod);
}

}  // namespace

hipError_t launch_lbfgs(const MultiFit *fits, int k_all, const double *out, int64_t ostride,
                        LbfgsState *states, int nfits, int m, double c1, double ftol,
                        hipStream_t stream, int polar, double rmin) {
    if (m != kLbfgsHist) return hipErrorInvalidValue;
    hipLaunchKernelGGL(lbfgs_kernel, dim3(nfits), dim3(64), 0, stream, fits, k_all, out, ostride, states, c1, ftol, polar,
                       rmin);
    return hipGetLastError();
}

}  // namespace pwa
