// Batched quasi-Newton minimisation of a bandwidth criterion over vech(L),
// H = L L^T, one independent problem per candidate (Sec. 5 names the PI and
// SCV selectors, Sec. 6 minimises them numerically without derivatives; here
// the exact gradients drive a BFGS inverse-Hessian update with a backtracking
// Armijo line search).
//
// The loop is a per-candidate state machine advanced by one update launch
// after each batched criterion evaluation: the evaluation takes the trial
// points xt of all candidates, the update reads their values and gradients,
// accepts or shortens the step and writes the next trial points.  A fixed
// number of evaluations is enqueued without host synchronisation, so a whole
// minimisation can be captured in a graph; finished candidates keep their
// point as the trial point (its evaluation is repeated and ignored).
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.h"
#include "minstep.h"

namespace kdefft {

namespace {

constexpr int MQ = 10;   // q = d(d+1)/2 <= 10 for d <= 4

__global__ void k_min_init(int64_t B, int q, const double* __restrict__ x0, double* __restrict__ xt,
                           int32_t* __restrict__ ist) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    for (int i = 0; i < q; ++i) xt[b * q + i] = x0[b * q + i];
    int32_t* is = ist + MIN_IS * b;
    is[0] = PH_START;
    is[1] = 0;                      // backtracks of the current line search
    is[2] = 0;                      // accepted steps
    is[3] = KDEFFT_MIN_RUNNING;     // outcome
    is[4] = 0;                      // accepted steps in a row without a decrease above rounding
}

// The update by itself, after a criterion that is not summed from lag items (PI).
template <int Q>
__global__ __launch_bounds__(64) void k_min_step(int64_t B, MinStep a, const double* __restrict__ ft, const double* __restrict__ gt) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    double g[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) g[i] = gt[b * Q + i];
    min_step<Q>(a, b, MinState<Q>(a, b), ft[b], g);
}

__global__ void k_min_final(int64_t B, int q, const double* __restrict__ st, const int32_t* __restrict__ ist,
                            double* __restrict__ x_out, double* __restrict__ f_out, int32_t* __restrict__ info) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const double* s = st + b * min_sw(q);
    for (int i = 0; i < q; ++i) x_out[b * q + i] = s[i];
    if (f_out) f_out[b] = s[3 * q + q * q];
    if (info) {
        info[2 * b] = ist[MIN_IS * b + 3];
        info[2 * b + 1] = ist[MIN_IS * b + 2];
    }
}

unsigned blocks_for(int64_t B) { return (unsigned)((B + 63) / 64); }

}  // namespace

int min_state_doubles(int q) { return min_sw(q); }
int min_state_ints() { return MIN_IS; }

hipError_t launch_min_init(int64_t B, int q, const double* x0, double* xt, int32_t* ist, hipStream_t s) {
    if (q < 1 || q > MQ) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_min_init, dim3(blocks_for(B)), dim3(64), 0, s, B, q, x0, xt, ist);
    return hipGetLastError();
}

hipError_t launch_min_step(int64_t B, int q, const MinStep& a, const double* ft, const double* gt, hipStream_t s) {
    const dim3 grid(blocks_for(B));
    switch (q) {
        case 1: hipLaunchKernelGGL(k_min_step<1>, grid, dim3(64), 0, s, B, a, ft, gt); break;
        case 3: hipLaunchKernelGGL(k_min_step<3>, grid, dim3(64), 0, s, B, a, ft, gt); break;
        case 6: hipLaunchKernelGGL(k_min_step<6>, grid, dim3(64), 0, s, B, a, ft, gt); break;
        case 10: hipLaunchKernelGGL(k_min_step<10>, grid, dim3(64), 0, s, B, a, ft, gt); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_min_final(int64_t B, int q, const double* st, const int32_t* ist, double* x_out, double* f_out,
                            int32_t* info, hipStream_t s) {
    if (q < 1 || q > MQ) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_min_final, dim3(blocks_for(B)), dim3(64), 0, s, B, q, st, ist, x_out, f_out, info);
    return hipGetLastError();
}

}  // namespace kdefft
