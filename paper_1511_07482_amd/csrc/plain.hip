// The paper's step 2 taken literally (Sec. 4): kernel values on the symmetric lag
// grid, stored in the circular zero-padded layout (lag l at index l mod P,
// Eq. (18)); steps 3 and 4 are in conv.hip.  And the assembly of the plain SCV
// criterion.
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "dev_kernels.h"
#include "internal.h"

namespace kdefft {

// Entries [first, first + nent) of the family at every lag of the slices l_0 < m
// (D = 1: the whole row), one lag per thread: its Gaussians are evaluated once
// for all entries.
template <int D, class Fun>
__global__ __launch_bounds__(256) void k_kgrid(double* __restrict__ out, kdefft_grid g, int64_t total,
                                               ParamBlock prm, int first, int nent) {
    Fun f;
    f.load(prm.v);
    for (int64_t e = blockIdx.x * 256LL + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        int64_t rem = e;
        double x[D];
        bool nz = true;
#pragma unroll
        for (int k = D - 1; k >= 0; --k) {
            const int p = (D > 1 && k == 0) ? (int)rem : (int)(rem & (g.P[k] - 1));
            rem >>= 31 - __clz(g.P[k]);
            int lag = 0;
            nz = nz && lag_of(p, g.M[k], g.P[k], &lag);
            x[k] = g.delta[k] * (double)lag;
        }
        double vals[Fun::NG];
        if (nz) {
            f.eval(x, vals);
        } else {
#pragma unroll
            for (int u = 0; u < Fun::NG; ++u) vals[u] = 0.0;
        }
#pragma unroll
        for (int u = 0; u < Fun::NG; ++u)
            if (u >= first && u < first + nent) out[(int64_t)(u - first) * total + e] = vals[u];
    }
}

static int64_t slice_values(const kdefft_grid& g, int m) {
    int64_t t = g.d > 1 ? m : g.P[0];
    for (int k = 1; k < g.d; ++k) t *= g.P[k];
    return t;
}

template <int D, class Fun>
static hipError_t kgrid_t(double* out, const kdefft_grid& g, int m, const ParamBlock& prm, int first, int nent,
                          hipStream_t s) {
    const int64_t total = slice_values(g, m);
    const int64_t b = (total + 255) / 256;
    hipLaunchKernelGGL((k_kgrid<D, Fun>), dim3((unsigned)(b > 16384 ? 16384 : b)), dim3(256), 0, s, out, g, total, prm,
                       first, nent);
    return hipGetLastError();
}

hipError_t launch_kgrid_psi(double* out, const kdefft_grid& g, int m, int r, const ParamBlock& prm, int first,
                            int nent, hipStream_t s) {
#define KG(DD, RR) if (g.d == DD && r == RR) return kgrid_t<DD, PsiFun<DD, RR>>(out, g, m, prm, first, nent, s);
    KG(1, 0) KG(1, 2) KG(1, 4) KG(1, 6) KG(1, 8)
    KG(2, 0) KG(2, 2) KG(2, 4) KG(2, 6) KG(2, 8)
    KG(3, 0) KG(3, 2) KG(3, 4) KG(3, 6)
    KG(4, 0) KG(4, 2) KG(4, 4)
#undef KG
    return hipErrorInvalidValue;
}

hipError_t launch_kgrid_scv(double* out, const kdefft_grid& g, int m, const ParamBlock& prm, int first, int nent,
                            hipStream_t s) {
    switch (g.d) {
        case 1: return kgrid_t<1, ScvPlainFun<1>>(out, g, m, prm, first, nent, s);
        case 2: return kgrid_t<2, ScvPlainFun<2>>(out, g, m, prm, first, nent, s);
        case 3: return kgrid_t<3, ScvPlainFun<3>>(out, g, m, prm, first, nent, s);
        case 4: return kgrid_t<4, ScvPlainFun<4>>(out, g, m, prm, first, nent, s);
        default: return hipErrorInvalidValue;
    }
}

// SCV(H) and d SCV / d vech(L) from the plain-path sums.
// sums[0] = n^-2 sum sum [phi_{S1} - 2 phi_{S2} + phi_{2G}], sums[1..q] the
// Hessian sums (already scaled).  fin: H^{-1} in slots [0,16), L in [16,32)
// (row stride 4), the first term n^-1 (4 pi)^{-d/2} |H|^{-1/2} in slot 32.
__global__ void k_scv_plain_final(const double* __restrict__ sums, ParamBlock fin, int d,
                                  double* __restrict__ out) {
    if (threadIdx.x != 0) return;
    const double* prm = fin.v;
    const double first = prm[32];
    double gH[4][4];
    int t = 1;
    for (int i = 0; i < d; ++i)
        for (int j = i; j < d; ++j) {
            const double v = -0.5 * first * prm[0 + i * 4 + j] + sums[t++];
            gH[i][j] = v;
            gH[j][i] = v;
        }
    out[0] = first + sums[0];
    // d SCV / d L = lower(2 gH L), vech by columns of the lower triangle
    int o = 1;
    for (int j = 0; j < d; ++j)
        for (int i = j; i < d; ++i) {
            double s = 0.0;
            for (int k = 0; k < d; ++k) s += gH[i][k] * prm[16 + k * 4 + j];
            out[o++] = 2.0 * s;
        }
}

hipError_t launch_scv_plain_final(const double* sums, const ParamBlock& fin, int d, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_scv_plain_final, dim3(1), dim3(64), 0, s, sums, fin, d, out);
    return hipGetLastError();
}

}  // namespace kdefft
