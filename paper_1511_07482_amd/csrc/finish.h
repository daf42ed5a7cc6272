// Assembly of the batched results from the per-item partial sums: psi
// entries, and criterion objective and gradient (fixed summation order).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dev_common.h"
#include "internal.h"

namespace kdefft {

// ------------------------------------------------------------------ small dense linear algebra (d <= 4)
// Cholesky A = L L^T of a symmetric d x d (row stride 4); false if not positive definite.
template <int D>
__device__ __forceinline__ static bool chol4(const double* A, double* L) {
#pragma unroll
    for (int i = 0; i < 16; ++i) L[i] = 0.0;
    bool ok = true;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        double s = A[j * 4 + j];
#pragma unroll
        for (int k = 0; k < j; ++k) s -= L[j * 4 + k] * L[j * 4 + k];
        ok = ok && (s > 0.0);
        const double ljj = sqrt(s > 0.0 ? s : 1.0);
        L[j * 4 + j] = ljj;
#pragma unroll
        for (int i = j + 1; i < D; ++i) {
            double t = A[i * 4 + j];
#pragma unroll
            for (int k = 0; k < j; ++k) t -= L[i * 4 + k] * L[j * 4 + k];
            L[i * 4 + j] = t / ljj;
        }
    }
    return ok;
}

// Inverse of L L^T from the lower factor L (row stride 4).
template <int D>
__device__ __forceinline__ static void chol_inv4(const double* L, double* Ainv) {
    double Li[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) Li[i] = 0.0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        Li[j * 4 + j] = 1.0 / L[j * 4 + j];
#pragma unroll
        for (int i = j + 1; i < D; ++i) {
            double s = 0.0;
#pragma unroll
            for (int k = j; k < i; ++k) s -= L[i * 4 + k] * Li[k * 4 + j];
            Li[i * 4 + j] = s / L[i * 4 + i];
        }
    }
#pragma unroll
    for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) {
            double s = 0.0;
#pragma unroll
            for (int k = (i > j ? i : j); k < D; ++k) s += Li[k * 4 + i] * Li[k * 4 + j];
            Ainv[i * 4 + j] = s;
        }
}

// Sum of the partial sums of candidate h, grid g over its chunks, by one
// wavefront: lane t takes chunks t, t+64, ... in order, then a fixed xor tree.
__device__ static double chunk_sum(const double* __restrict__ partial, int64_t h, int64_t nchunks, int ng, int g) {
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    for (int64_t c = lane; c < nchunks; c += 64) s += partial[(h * nchunks + c) * ng + g];
    return wave_sum(s);
}

// Sums over candidate h's count items (partial sums of ng values per item) of
// its first NG grids (a grid from ng on gives 0) into T[0, NG), and of the first
// grid of candidate c (if c >= 0) into T[NG], by one wavefront in the same fixed
// order as chunk_sum; all loads and trees are in flight together.
template <int NG>
__device__ __forceinline__ static void item_sums(const double* __restrict__ partial, int64_t h, int64_t c,
                                                 int64_t count, int ng, double* T) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int g = 0; g <= NG; ++g) T[g] = 0.0;
    const double* own = partial + h * count * ng;
    const double* other = c >= 0 ? partial + c * count * ng : own;
    for (int64_t i = lane; i < count; i += 64) {
#pragma unroll
        for (int g = 0; g < NG; ++g) T[g] += own[i * ng + (g < ng ? g : 0)];
        T[NG] += other[i * ng];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int g = 0; g <= NG; ++g) T[g] += __shfl_xor(T[g], off, 64);
#pragma unroll
    for (int g = 0; g <= NG; ++g) T[g] = (g == NG ? c >= 0 : g < ng) ? T[g] : 0.0;
}

// Slots 0..63 of a parameter block, one per lane (loaded with the sums' loads,
// not after them).
struct ParamLanes {
    double v;
    __device__ __forceinline__ explicit ParamLanes(const double* __restrict__ p) : v(p[threadIdx.x & 63]) {}
    __device__ __forceinline__ double operator[](int slot) const {   // wavefront-uniform
        const long long b = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_readlane((int)b, slot), hi = __builtin_amdgcn_readlane((int)(b >> 32), slot);
        return __longlong_as_double((long long)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo));
    }
};

// Criterion assembly for a candidate (p: its parameter block, T: its sums over
// the lags), by a whole wavefront.  kind: FUN_SCV_OBJ or FUN_ETA* (objective only), FUN_SCV_OBJGRAD
// (objective + gradient), FUN_SCV_GRAD (adjoint: gradient scaled by gscale).
// cst is the constant term added to the objective (the SCV phi_{2G} sum, else
// 0).  Returns the objective; gv: the gradient in vech(L) order, if kind has one.
template <int D>
__device__ __forceinline__ static double crit_finish(int kind, const double* T, const ParamLanes& p,
                                                     double cst, double gscale, bool want_grad, double* gv) {
    constexpr int d = D;
    const bool sing = p[S_SING] != 0.0;
    const double nan = __longlong_as_double(0x7ff8000000000000LL);
    // closed-form term: proportional to |H|^{-1/2} for every criterion with a
    // gradient, so its matrix gradient is -1/2 first H^{-1}
    const double t0 = p[S_FIRST], scale = p[S_SCALE];
    const double obj = sing ? nan : t0 + T[0] * scale + cst;
    if (!want_grad) return obj;
    double L[16], Hinv[16], gH[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) L[i] = p[S_L + i];
    chol_inv4<D>(L, Hinv);
    const bool both = kind == FUN_SCV_OBJGRAD;   // T[0] is the objective's sum
    int t = 0;
#pragma unroll
    for (int i = 0; i < d; ++i)
#pragma unroll
        for (int j = i; j < d; ++j) {
            const double v = -0.5 * t0 * Hinv[i * 4 + j] + (both ? T[t + 1] : T[t]) * scale;
            ++t;
            gH[i * 4 + j] = v;
            gH[j * 4 + i] = v;
        }
    int o = 0;
#pragma unroll
    for (int j = 0; j < d; ++j)
#pragma unroll
        for (int i = j; i < d; ++i) {
            double s = 0.0;
#pragma unroll
            for (int k = j; k < d; ++k) s += gH[i * 4 + k] * L[k * 4 + j];
            gv[o++] = sing ? nan : 2.0 * s * gscale;
        }
    return obj;
}

__device__ __forceinline__ static void* slot_ptr(double v) {
    return reinterpret_cast<void*>(static_cast<uintptr_t>(__double_as_longlong(v)));
}

}  // namespace kdefft
