// Start and result of fits whose L-BFGS states live on the device: start vectors
// come from, and the few results go to, small records in mapped host memory, so a
// state (28.6 KB, nearly all history) never crosses the bus.  24 fits of
// four iterations: 4.1 and 3.0 us of a call, which went from 622 to 549 us with the
// copies of whole states from and to pageable memory gone.
#include "internal.hpp"

namespace pwa {
namespace {

constexpr int kStateThreads = 256;

// Fit blockIdx.x: its state cleared (phase 0) with the start's trial point.
__global__ __launch_bounds__(kStateThreads) void fit_start_kernel(LbfgsState *states, const FitStart *start) {
    const int f = blockIdx.x, i = threadIdx.x;
    LbfgsState *st = states + f;
    constexpr int kWords = sizeof(LbfgsState) / sizeof(double);
    static_assert(sizeof(LbfgsState) % sizeof(double) == 0 && kLbfgsMaxN <= kStateThreads, "state layout");
    const bool mine = i < kLbfgsMaxN;
    const double xt = mine ? start[f].xt[i] : 0.0, vt = mine ? start[f].vt[i] : 0.0;
    double *w = reinterpret_cast<double *>(st);
    for (int j = i; j < kWords; j += kStateThreads) w[j] = 0.0;
    __syncthreads();
    if (mine) {
        st->xt[i] = xt;
        st->vt[i] = vt;
    }
}

// Before the first evaluation the accepted point is the start point.
__global__ __launch_bounds__(kStateThreads) void fit_result_kernel(const LbfgsState *states, FitResult *result) {
    const int f = blockIdx.x, i = threadIdx.x;
    const LbfgsState *st = states + f;
    const int started = st->phase != 0;
    if (i < kLbfgsMaxN) result[f].x[i] = started ? st->x[i] : st->xt[i];
    if (i == 0) {
        result[f].f = st->f;
        result[f].started = started;
        result[f].status = st->status;
        result[f].iter = st->iter;
    }
}

}  // namespace

hipError_t launch_fit_start(LbfgsState *states, const FitStart *start, int nfits, hipStream_t stream) {
    hipLaunchKernelGGL(fit_start_kernel, dim3(nfits), dim3(kStateThreads), 0, stream, states, start);
    return hipGetLastError();
}

hipError_t launch_fit_result(const LbfgsState *states, FitResult *result, int nfits, hipStream_t stream) {
    hipLaunchKernelGGL(fit_result_kernel, dim3(nfits), dim3(kStateThreads), 0, stream, states, result);
    return hipGetLastError();
}

}  // namespace pwa
