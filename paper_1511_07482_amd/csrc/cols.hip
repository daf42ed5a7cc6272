// Column walk (cols.h): geometry, and the launchers of the SCV families.
#include "cols.h"

#include <algorithm>

namespace kdefft {

// Resident blocks on the current device: the kernels' launch bounds ask for
// about four blocks of 256 threads per CU.
static int cols_slots() {
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
// the 256-candidate SCV call took 53, 59, 67 us instead of 48).  d >= 3: groups
// of axis-0 lags (a power of two from 8 on, so that a group's planes stay within
// about 2 MB), split further when the candidates are few; psi, whose parts one
// block adds up, takes at most 256 of them.
ColGeom cols_geom(const kdefft_grid& g, int64_t ncand, int ng, bool scv, int64_t max_chunks) {
    ColGeom geo{};
    for (int k = 0; k < 4; ++k) {
        geo.M[k] = k < g.d ? g.M[k] : 1;
        geo.P[k] = k < g.d ? g.P[k] : 1;
    }
    const int64_t slots = cols_slots(), steps = cols_steps(g);
    const int d = g.d;
    int64_t per = (slots + ncand - 1) / ncand;
    if (per > 1 && ncand * per > slots + slots / 8) per = slots / ncand > 1 ? slots / ncand : 1;
    if (per > steps) per = steps;
    if (!scv && per > 256) per = 256;
    // a batch that fits the fixed scratch of the call without a workspace keeps fitting it
    const int64_t room = scv ? ((int64_t)KDEFFT_NOALLOC_BYTES - (1 << 19)) / (8 * ncand) - PRM : (int64_t)1 << 40;
    geo.n0 = 1;
    if (d >= 3) {
        const int64_t slice = 8LL * g.P[d - 1] * g.P[d - 2] * (d == 4 ? g.P[1] : 1);
        int n0 = 1;
        while (2 * n0 <= g.M[0] && (n0 < 8 || g.M[0] * slice > n0 * (2LL << 20))) n0 *= 2;
        while (n0 > 1 && (n0 * ng > room || n0 > max_chunks)) n0 /= 2;
        int64_t nsub = (per + n0 - 1) / n0;
        if (nsub > 1 && n0 * nsub * ng > room) nsub = 1;
        if (n0 * nsub > max_chunks) nsub = std::max<int64_t>(max_chunks / n0, 1);
        geo.n0 = n0;
        geo.nchunks = n0 * nsub;
        return geo;
    }
    while (per > 1 && per * ng > room) per /= 2;
    geo.nchunks = std::min(per, std::max<int64_t>(max_chunks, 1));
    return geo;
}

int64_t cols_blocks(int64_t nitems, int grid_blocks) {
    const int64_t blocks = grid_blocks > 0 ? grid_blocks : (grid_blocks == 0 ? cols_slots() : nitems);
    return blocks < nitems ? blocks : nitems;
}

template <int D, int MODE>
static hipError_t run_cols(const ColGeom& geo, const ScvSetup& setup, int64_t nitems, double* partial, int gb,
                           hipStream_t s) {
    const dim3 grid((unsigned)cols_blocks(nitems, gb)), nt(COL_NT);
    if constexpr (D >= 2) {
        if (geo.P[D - 2] < 16) {
            hipLaunchKernelGGL((k_cols_scv<D, MODE, true>), grid, nt, 0, s, geo, setup, nitems, partial);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_cols_scv<D, MODE, false>), grid, nt, 0, s, geo, setup, nitems, partial);
    return hipGetLastError();
}

template <int D>
static hipError_t run_cols_mode(int kind, const ColGeom& geo, const ScvSetup& setup, int64_t nitems, double* partial,
                                int gb, hipStream_t s) {
    switch (kind) {
        case FUN_SCV_OBJ: return run_cols<D, 0>(geo, setup, nitems, partial, gb, s);
        case FUN_SCV_OBJGRAD: return run_cols<D, 1>(geo, setup, nitems, partial, gb, s);
        case FUN_SCV_GRAD: return run_cols<D, 2>(geo, setup, nitems, partial, gb, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_cols_scv(int kind, int d, const ColGeom& geo, const ScvSetup& setup, int64_t nitems,
                           double* partial, int gb, hipStream_t s) {
    if (nitems < 1) return hipSuccess;
    switch (d) {
        case 1: return run_cols_mode<1>(kind, geo, setup, nitems, partial, gb, s);
        case 2: return run_cols_mode<2>(kind, geo, setup, nitems, partial, gb, s);
        case 3: return run_cols_mode<3>(kind, geo, setup, nitems, partial, gb, s);
        case 4: return run_cols_mode<4>(kind, geo, setup, nitems, partial, gb, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kdefft
