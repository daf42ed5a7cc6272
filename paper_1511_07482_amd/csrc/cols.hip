// Launchers of the column walk (cols.h).
#include "cols.h"

namespace kdefft {

// Resident blocks on the current device: the kernels' launch bounds ask for
// four blocks of 256 threads per CU.
int cols_slots() {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    if (cus[dev] <= 0) {
        int c = 0;
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c < 1) c = 256;
        cus[dev] = c;
    }
    return cus[dev] * 4;
}

// Block steps (16 units) of one candidate whose whole lag box is live.
static int64_t cols_steps(const kdefft_grid& g) {
    const int d = g.d;
    if (d == 1) return 1;
    const int N = g.P[d - 1], lx = g.M[d - 1] - 1, lw = g.M[d - 2] - 1;
    const bool small = g.P[d - 2] < 16;
    int64_t u = N <= 16 ? 1 : lx / 16 + 1 + (lx + 15) / 16;
    u *= small ? 1 : col_segs(d, lw);
    if (d >= 3) u *= g.M[0];
    if (d == 4) u *= 2 * g.M[1] - 1;
    return (u + 15) / 16;
}

// d = 2: one round of the resident blocks (an item's set-up and reductions are
// several microseconds of latency: with two, three, four rounds of smaller items
// the 256-candidate call took 53, 59, 67 us instead of 48).  d >= 3: groups of
// axis-0 lags (a power of two from 8 on, so that a group's planes stay within
// about 2 MB), split further when the candidates are few.
void cols_geom(const kdefft_grid& g, int64_t ncand, RowGeom* geo) {
    const int64_t slots = cols_slots(), steps = cols_steps(g);
    const int d = g.d, ng = 1 + d * (d + 1) / 2;
    int64_t per = (slots + ncand - 1) / ncand;
    if (per > 1 && ncand * per > slots + slots / 8) per = slots / ncand > 1 ? slots / ncand : 1;
    if (per > steps) per = steps;
    // a batch that fits the fixed scratch of the call without a workspace keeps fitting it
    const int64_t room = ((int64_t)KDEFFT_NOALLOC_BYTES - (1 << 19)) / (8 * ncand) - PRM;
    geo->n0 = 1;
    if (d >= 3) {
        const int64_t slice = 8LL * g.P[d - 1] * g.P[d - 2] * (d == 4 ? g.P[1] : 1);
        int n0 = 1;
        while (2 * n0 <= g.M[0] && (n0 < 8 || g.M[0] * slice > n0 * (2LL << 20))) n0 *= 2;
        while (n0 > 1 && n0 * ng > room) n0 /= 2;
        int64_t nsub = (per + n0 - 1) / n0;
        if (nsub > 1 && n0 * nsub * ng > room) nsub = 1;
        geo->n0 = n0;
        geo->nchunks = n0 * nsub;
        return;
    }
    while (per > 1 && per * ng > room) per /= 2;
    geo->nchunks = per;
}

template <int D, int MODE>
static hipError_t run_cols(const RowGeom& geo, int64_t nitems, double* partial, int grid_blocks, hipStream_t s) {
    int64_t blocks = grid_blocks > 0 ? grid_blocks : (grid_blocks == 0 ? cols_slots() : nitems);
    if (blocks > nitems) blocks = nitems;
    if (blocks < 1) return hipSuccess;
    const dim3 grid((unsigned)blocks), nt(COL_NT);
    if constexpr (D >= 2) {
        if (geo.P[D - 2] < 16) {
            hipLaunchKernelGGL((k_cols_scv<D, MODE, true>), grid, nt, 0, s, geo, nitems, partial);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_cols_scv<D, MODE, false>), grid, nt, 0, s, geo, nitems, partial);
    return hipGetLastError();
}

template <int D>
static hipError_t run_cols_mode(int kind, const RowGeom& geo, int64_t nitems, double* partial, int gb, hipStream_t s) {
    switch (kind) {
        case FUN_SCV_OBJ: return run_cols<D, 0>(geo, nitems, partial, gb, s);
        case FUN_SCV_OBJGRAD: return run_cols<D, 1>(geo, nitems, partial, gb, s);
        case FUN_SCV_GRAD: return run_cols<D, 2>(geo, nitems, partial, gb, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_cols_scv(int kind, const RowGeom& geo, int64_t nitems, double* partial, int grid_blocks,
                           hipStream_t s) {
    switch (geo.d) {
        case 1: return run_cols_mode<1>(kind, geo, nitems, partial, grid_blocks, s);
        case 2: return run_cols_mode<2>(kind, geo, nitems, partial, grid_blocks, s);
        case 3: return run_cols_mode<3>(kind, geo, nitems, partial, grid_blocks, s);
        case 4: return run_cols_mode<4>(kind, geo, nitems, partial, grid_blocks, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kdefft
