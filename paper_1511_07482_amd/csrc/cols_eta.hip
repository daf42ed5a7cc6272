// Column walk (cols.h): launchers of the scalar eta_r families of low order.
#include "cols.h"

namespace kdefft {

// The sums of order 2r need C(d + 2r - 1, 2r) accumulators per Gaussian and
// lose digits where the contraction cancels, more with every order: r <= 2 (d =
// 4, whose r = 2 would take 70 accumulators: r <= 1); the row walk of rows_impl.h
// serves the others.
bool cols_eta_ok(int d, int r) { return r <= (d == 4 ? 1 : 2); }

template <int D, int NGS, int R>
static hipError_t run_eta(const ColGeom& geo, const ScvSetup& setup, int64_t nitems, double* partial, int gb,
                          hipStream_t s) {
    const dim3 grid((unsigned)cols_blocks(nitems, gb)), nt(COL_NT);
    if constexpr (D >= 2) {
        if (geo.P[D - 2] < 16) {
            hipLaunchKernelGGL((k_cols_eta<D, NGS, R, true>), grid, nt, 0, s, geo, setup, nitems, partial);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_cols_eta<D, NGS, R, false>), grid, nt, 0, s, geo, setup, nitems, partial);
    return hipGetLastError();
}

hipError_t launch_cols_eta(int kind, int d, int r, const ColGeom& geo, const ScvSetup& setup, int64_t nitems,
                           double* partial, int gb, hipStream_t s) {
    if (nitems < 1) return hipSuccess;
    const int ngs = kind == FUN_ETA1 ? 1 : 2;
#define ETA(DD, RR)                                                                                  \
    if (d == DD && r == RR)                                                                          \
        return ngs == 1 ? run_eta<DD, 1, RR>(geo, setup, nitems, partial, gb, s)                     \
                        : run_eta<DD, 2, RR>(geo, setup, nitems, partial, gb, s);
    ETA(1, 0) ETA(1, 1) ETA(1, 2)
    ETA(2, 0) ETA(2, 1) ETA(2, 2)
    ETA(3, 0) ETA(3, 1) ETA(3, 2)
    ETA(4, 0) ETA(4, 1)
#undef ETA
    return hipErrorInvalidValue;
}

}  // namespace kdefft
