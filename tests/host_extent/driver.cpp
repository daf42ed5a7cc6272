// Launch extents of the batched criteria against the workspace they are given,
// over thin and long grids, every kernel family and variant, and batches whose
// candidates share the device unevenly; and the column walk's unit numbers, taken
// apart as the kernel does, up to the largest a part can have.  Host only:
// nothing is launched.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "internal.h"

using namespace kdefft;

static long long fails = 0, checked = 0;

static kdefft_grid shape(int d, const int* M) {
    kdefft_grid g{};
    g.d = d;
    for (int k = 0; k < 4; ++k) {
        g.M[k] = k < d ? M[k] : 1;
        g.P[k] = k < d ? 4 : 1;
        while (k < d && g.P[k] < 2 * g.M[k]) g.P[k] *= 2;
        g.delta[k] = 1.0;
    }
    return g;
}

static void check(const kdefft_grid& g, int64_t B) {
    const int64_t room = crit_room(g, B);
    const int n_ds[3] = {0, 1, KDEFFT_MAX_BATCH_DS};   // constant-term candidates of the launch
    for (int kind = FUN_SCV_OBJ; kind <= FUN_ETA2; ++kind) {
        const bool eta = kind == FUN_ETA1 || kind == FUN_ETA2;
        for (int variant = 0; variant < ROW_VARIANTS; ++variant)
            for (int r = eta ? 1 : 0; r <= (eta ? 3 : 0); r += 2)
                for (int e : n_ds) {
                    if (eta && (e || (variant != 3 && variant != 4))) continue;
                    const int64_t nc = B + e;
                    const CritWalk w = crit_walk(g, kind, r, variant, nc, room);
                    const int64_t used = nc * w.nchunks * ng_of(kind, g.d, 2);
                    // what the launch visits: all rows, or whole groups of axis-0 lags
                    const bool whole = w.cols ? w.nchunks >= 1 && w.col.n0 >= 1 && w.nchunks % w.col.n0 == 0
                                              : w.row.chunk * w.nchunks >= w.row.nrows;
                    ++checked;
                    if (used > room || !whole) {
                        if (fails++ < 5)
                            std::printf("d=%d M=[%d,%d,%d,%d] B=%lld +%d kind %d variant %d r %d: %lld of %lld doubles\n",
                                        g.d, g.M[0], g.M[1], g.M[2], g.M[3], (long long)B, e, kind, variant, r,
                                        (long long)used, (long long)room);
                    }
                }
    }
}

// Every u around a multiple of d of a candidate of `total` units.
template <int D>
static void check_quotients(int d, int total) {
    const ColRecip<D> rd = 1 / (ColRecip<D>)d;
    for (int64_t m = 0; m < total; m += d)
        for (int64_t u = m > 0 ? m - 1 : 0; u <= m + 1 && u < total; ++u) {
            ++checked;
            if (col_quot((int)u, rd) != u / d && fails++ < 5)
                std::printf("d=%d unit %lld of %d: quotient by %d\n", D, (long long)u, total, d);
        }
}

// The largest number of units a launch of dimension d can ask for (prod P <=
// 2^30, one axis-0 group), as cols.h counts them.
static int64_t most_units(int d) {
    int64_t most = 0;
    for (int n = 2; n <= 2048; n *= 2)             // nodes of the last axis; P = 2 n
        for (int w = 2; w <= 2048; w *= 2)         // of the walked one
            for (int a = d > 2 ? 2 : 1; a <= (d > 2 ? 2048 : 1); a *= 2)
                for (int b = d > 3 ? 2 : 1; b <= (d > 3 ? 2048 : 1); b *= 2)
                    for (int e = 0; e < 2; ++e) {   // just past half a padded axis, and filling it
                        const int64_t P = 4LL * n * w * (d > 2 ? 2 * a : 1) * (d > 3 ? 2 * b : 1);
                        if (P > (1LL << 30)) continue;
                        const int lx = (e ? n : n / 2 + 1) - 1, lw = (e ? w : w / 2 + 1) - 1;
                        int64_t u = 2 * n <= 16 ? 1 : lx / 16 + 1 + (lx + 15) / 16;
                        const int side = d == 2 || lw < 32 ? 0 : (lw - 32) / 64 + 1;
                        u *= 2 * w < 16 ? 1 : d == 2 ? lw / 64 + 1 : 2 * side + 1;
                        u *= (d > 2 ? a : 1) * (d > 3 ? 2LL * b - 1 : 1);
                        if (u > most) most = u;
                    }
    return most;
}

int main() {
    for (int d : {1, 2, 3, 5, 7, 31, 32, 33, 63, 129, 257, 1000, 4095}) {
        check_quotients<2>(d, (int)most_units(2));
        check_quotients<3>(d, (int)most_units(3));
        check_quotients<4>(d, (int)most_units(4));
    }
    if (most_units(3) >= 1 << 21 || most_units(4) < 1 << 22) {
        ++fails;
        std::printf("units: %lld at d = 3, %lld at d = 4\n", (long long)most_units(3), (long long)most_units(4));
    }
    // thin first axes beside long ones, batches around a whole number per resident block
    for (int m0 = 2; m0 <= 8; ++m0)
        for (int m1 : {2, 17, 155, 372, 511}) {
            const int M[4] = {m0, m1, 1, 1};
            const kdefft_grid g = shape(2, M);
            for (int64_t B = 1; B <= 1200; B += B < 32 ? 1 : 7) check(g, B);
            for (int64_t B : {256, 266, 512, 522, 569}) check(g, B);
        }
    // the benchmark's shape (as its tuner runs it), and shapes of each dimension
    const int listed[][5] = {{2, 256, 256, 1, 1}, {1, 1000, 1, 1, 1}, {3, 17, 2, 121, 1}, {3, 804, 424, 138, 1},
                             {3, 64, 64, 64, 1},  {4, 32, 32, 32, 32}, {4, 64, 2048, 2, 256}};
    for (const auto& l : listed)
        for (int64_t B : {1, 6, 101, 256, 498, 1024, 24407}) check(shape(l[0], l + 1), B);
    std::mt19937 rng(7);
    for (int t = 0; t < 4000; ++t) {
        const int d = 1 + (int)(rng() % 4);
        const int most[5] = {0, 2048, 600, 150, 40};
        int M[4] = {1, 1, 1, 1};
        for (int k = 0; k < d; ++k) M[k] = 2 + (int)(rng() % (rng() % 2 ? 7 : most[d] - 1));
        check(shape(d, M), 1 + (int64_t)(rng() % (rng() % 2 ? 1200 : 40000)));
    }
    std::printf("%lld checks, %lld failures\n", checked, fails);
    if (fails == 0) std::printf("ok\n");
    return fails != 0;
}
