// Column walk (cols.h): launchers of the psi_r functionals.
#include "cols.h"

namespace kdefft {

template <int D, int R>
static hipError_t run_psi(const ColGeom& geo, const PsiBatchArgs& a, int gb, double* prm, double* partial,
                          double* psi, hipStream_t s) {
    const int64_t nitems = a.n_ds * geo.nchunks;
    const dim3 grid((unsigned)cols_blocks(nitems, gb)), nt(COL_NT);
    bool small = false;
    if constexpr (D >= 2) {
        small = geo.P[D - 2] < 16;
        if (small) hipLaunchKernelGGL((k_cols_psi<D, R, true>), grid, nt, 0, s, geo, a, nitems, prm, partial);
    }
    if (!small) hipLaunchKernelGGL((k_cols_psi<D, R, false>), grid, nt, 0, s, geo, a, nitems, prm, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_cols_psi_final<D, R>), dim3((unsigned)a.n_ds), nt, 0, s, partial, geo.nchunks, prm, psi);
    return hipGetLastError();
}

hipError_t launch_cols_psi(const ColGeom& geo, const PsiBatchArgs& a, int gb, double* prm, double* partial,
                           double* psi, hipStream_t s) {
    if (a.n_ds < 1) return hipSuccess;
#define PSI(DD, RR) if (a.d == DD && a.r == RR) return run_psi<DD, RR>(geo, a, gb, prm, partial, psi, s);
    PSI(1, 0) PSI(1, 2) PSI(1, 4) PSI(1, 6) PSI(1, 8)
    PSI(2, 0) PSI(2, 2) PSI(2, 4) PSI(2, 6) PSI(2, 8)
    PSI(3, 0) PSI(3, 2) PSI(3, 4) PSI(3, 6)
    PSI(4, 0) PSI(4, 2) PSI(4, 4)
#undef PSI
    return hipErrorInvalidValue;
}

}  // namespace kdefft
