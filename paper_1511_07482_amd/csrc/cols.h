// Column walk: the lag-domain sums sum_l k(l) A(l) of the batched criteria,
// walked along axis D-2 of the lag array with 16 neighbouring lags of the last
// axis on the 16 lanes of a group (D = 1: one lag per lane, no walk).
//
// Coordinates.  With S = L L^T in the axis order (0..D-3, D-1, D-2) and
// y = L^{-1} x, every Gaussian of the family is c exp(-|y|^2 / 2), D^{(x)2} phi =
// L^{-T} (y y^T - I) L^{-1} phi, and only the last component y_w changes along
// the walked axis (by u per lag).  A column (fixed lags of the other axes)
// therefore costs the moments m_p = sum w y_w^p, w = exp(-|y|^2 / 2) A; the
// products with the fixed components are added once per column, and L^{-1} is
// applied once per work item.
//
// Along a column, with y the walked component at a run's first row,
//   exp(-(y + u t)^2 / 2) = e r^t g_t,  e = exp(-y^2 / 2), r = exp(-u y),
//   g_t = exp(-u^2 t^2 / 2) (the same for every column: computed once per item),
// so a run of RUN = 8 rows is a polynomial in r with the coefficients a_t g_t:
// one Horner scheme and its two nested ones give sum w, sum s w and
// sum s(s+1)/2 w (s = t + 1) in four operations per lag and Gaussian.  The next
// run starts at e s and r exp(-8 u^2), its s is s exp(-64 u^2) (s = r^8 g_8, from the
// start on its own: as a power of each run's r it would take eight times that
// run's roundings); a column is walked in segments of
// SEG rows, each started with exponentials.  The walked component of each run is
// formed from its lag, not added up: the roundings of the far end would stay in
// it (d = 3 and 4 gradients 6.5e-15 and 1.2e-14 off, so 3.6e-15 and 5.1e-15).  The constants that carry a walk
// on are common to all columns, so their rounding would not average out (with
// plain doubles 1.5e-14 of the d = 3, 4 results): they are kept as two doubles.
// Errors of whole results against extended precision, 2-norm relative, mean of 12
// samples, s as a power of r -> s by itself (a row walk of the same sums): d = 3,
// M = 64 SCV objective 2.9e-15 -> 1.1e-15 (1.3e-15), gradient 1.7e-15 -> 1.1e-15
// (0.9e-15), psi_4 3.1e-14 -> 1.4e-14 (0.7e-14; one with the components' low
// parts too), psi_2 2.7e-15 -> 1.0e-15 (5.2e-15); d = 2, M = 203 gradient 2.1e-15 ->
// 1.7e-15 (3.5e-15).
//
// Bound: FP64 issue (d = 4), the latency of an item's set-up and reductions
// (few candidates).  16 lanes x 8 bytes are one cache line, so a wavefront's
// load touches four lines; a row-wise walk (one lane per row run) touches 64
// and folds 25 flops per Hessian entry into every run.  Whole SCV
// objective-and-gradient call, replayed: d = 2, M = 256, 256 candidates 53.1 ->
// 37.0 us, 4 candidates 23.6 -> 16.2 us; d = 3, M = 64, 64 candidates 150 ->
// 57 us; d = 4, M = 32, four datasets of 64 candidates 3618 -> 906 us (row walk
// -> column walk; 979 before the walk was cut to the lags that the data reach).
//
// Live set: a lag is walked when its first Gaussian is at or above the cut of
// its peak (LOG_REL_CUT).  The first Gaussian is the widest of its family
// (2H + 2G against H + 2G, 2H against H), so it bounds the others; the walk
// enumerates the box around its ellipsoid, cut to the lags the data reach (the
// grid is wider by the kernel's padding: the autocorrelation is zero there),
// and each column's interval is found in closed form.  Every start is at most RUN - 1 lags before a column's live
// interval, so with u^2 < log 2 no value under- or overflows; a kernel narrower
// than that is evaluated lag by lag.
#pragma once

#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "dev_kernels.h"
#include "finish.h"
#include "internal.h"
#include "params.h"
#include "rows_impl.h"

namespace kdefft {

constexpr int COL_RUN = 8;    // rows per run
// Rows per segment: one start with exponentials each (at d = 2, where the columns
// are few, 32 rows measured 27.5 and 25.0 us for 64 candidates at M = 256 and 101
// at M = 203, 64 rows 24.2 and 22.5; 256 candidates the same).
constexpr int COL_SEG = 64;
// Segments of an axis with lags up to lw: D = 2 from lag 0 on (half set);
// D >= 3 around lag 0, segment s of [-n, n] covering the rows from
// COL_SEG * s - COL_SEG / 2.
__host__ __device__ constexpr int col_side_segs(int D, int lw) {
    return D == 2 || lw < COL_SEG / 2 ? 0 : (lw - COL_SEG / 2) / COL_SEG + 1;
}
__host__ __device__ constexpr int col_segs(int D, int lw) {
    return D == 2 ? lw / COL_SEG + 1 : 2 * col_side_segs(D, lw) + 1;
}
constexpr int COL_NT = 256;
static_assert(COL_RUN == 8, "the run's powers and tables are written for 8 rows");

// Axis at position p of the walk order: the walked axis D-2 last, the last
// axis (the lanes) before it.
__host__ __device__ constexpr int col_axis(int D, int p) {
    return D == 1 ? 0 : (p < D - 2 ? p : (p == D - 2 ? D - 1 : D - 2));
}
__host__ __device__ constexpr int col_pos(int D, int axis) {
    for (int p = 0; p < D; ++p)
        if (col_axis(D, p) == axis) return p;
    return 0;
}
__host__ __device__ constexpr int tri(int i, int j) { return i * (i + 1) / 2 + j; }

// One Gaussian of an item: L^{-1} in walk order, scaled by the grid spacing (ld:
// y = ld lag, packed lower) and plain (li), normal constant, run tables.
template <int D>
struct ColGauss {
    double ld[D * (D + 1) / 2];
    double li[D * D];         // (square, zero above the diagonal)
    double c;
    double gt[COL_RUN];   // exp(-u^2 t^2 / 2), t < RUN
    // exp(-RUN u^2), exp(-RUN^2 u^2 / 2) and exp(-RUN^2 u^2), as high and low parts
    double h[2], g8[2], h8[2];
};

// An item's parameters, in LDS.
template <int D, int NGS>
struct ColItem {
    ColGauss<D> g[NGS];
    double sign;
    const double* A;
    int lm[4];   // largest |lag| at each position of the walk order
};

// Factor A (row stride 4, walk order) in place of its inverse: li = L^{-1} packed
// lower, *det = |A|^{-1/2}; false if A is not positive definite (then the
// identity, whose results the caller discards).  One reciprocal root per pivot:
// the set-up is one lane's serial chain at the start of every item.
template <int D>
__device__ __forceinline__ bool col_factor(double (&A)[D][D], bool bad, double* li, double* det) {
    double r[D];
    bool ok = !bad;
#pragma unroll
    for (int j = 0; j < D; ++j) {
        double s = A[j][j];
#pragma unroll
        for (int k = 0; k < j; ++k) s = fma(-A[j][k], A[j][k], s);
        ok = ok && s > 0.0;
        r[j] = rsqrt(s > 0.0 ? s : 1.0);
#pragma unroll
        for (int i = j + 1; i < D; ++i) {
            double t = A[i][j];
#pragma unroll
            for (int k = 0; k < j; ++k) t = fma(-A[i][k], A[j][k], t);
            A[i][j] = t * r[j];
        }
    }
    *det = 1.0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        li[tri(i, i)] = ok ? r[i] : 1.0;
        *det *= li[tri(i, i)];
#pragma unroll
        for (int j = 0; j < i; ++j) {
            double s = 0.0;
#pragma unroll
            for (int k = j; k < i; ++k) s = fma(-A[i][k], li[tri(k, j)], s);
            li[tri(i, j)] = ok ? s * r[i] : 0.0;
        }
    }
    return ok;
}

// 2^(j/32) as high and low parts.
static __device__ const double2 COL_EXP2[32] = {
    {1.0, 0.0}, {1.0218971486541166, 5.109225028973444e-17},
    {1.0442737824274138, 8.551889705537965e-17}, {1.0671404006768237, -7.899853966841582e-17},
    {1.0905077326652577, -3.046782079812471e-17}, {1.1143867425958924, 1.0410278456845571e-16},
    {1.1387886347566916, 8.912812676025408e-17}, {1.1637248587775775, 3.8292048369240935e-17},
    {1.189207115002721, 3.982015231465646e-17}, {1.215247359980469, -7.712630692681488e-17},
    {1.241857812073484, 4.658027591836937e-17}, {1.2690509571917332, 2.667932131342186e-18},
    {1.2968395546510096, 2.5382502794888315e-17}, {1.3252366431597413, -2.8587312100388614e-17},
    {1.3542555469368927, 7.70094837980299e-17}, {1.383909881963832, -6.770511658794786e-17},
    {1.4142135623730951, -9.667293313452913e-17}, {1.4451808069770467, -3.0237581349939873e-17},
    {1.4768261459394993, -3.483994556892796e-17}, {1.5091644275934228, -1.016455327754295e-16},
    {1.5422108254079407, 7.949834809697621e-17}, {1.5759808451078865, -1.0136916471278304e-17},
    {1.6104903319492543, 2.4707192569797888e-17}, {1.645755478153965, -1.0125679913674773e-16},
    {1.681792830507429, 8.199010020581497e-17}, {1.718619298122478, -1.851380418263111e-17},
    {1.7562521603732995, 2.960140695448873e-17}, {1.7947090750031072, 1.8227458427912087e-17},
    {1.8340080864093424, 3.283107224245627e-17}, {1.8741676341103, -6.122763413004143e-17},
    {1.9152065613971474, -1.0619946056195963e-16}, {1.9571441241754002, 8.960767791036668e-17}};

// exp(x + xl) for a small correction xl, by the table-driven method of P. T. P.
// Tang (ACM Trans. Math. Softw. 15, 1989): x = (32 k + j) log 2 / 32 + r,
// |r| < 0.011, 2^(j/32) from the table (a copy in LDS), the series of exp(r) to
// r^6.  One rounding of any weight, so the error is that of one rounding and
// without a bias; a bias of the start's r would be multiplied by the lags
// walked (the library's exp left 2e-15 of a d = 3 sum, this 3e-16) -- and it
// takes half the instructions.
__device__ __forceinline__ double2 col_exp2(double x, double xl, const double2* tab, int* k) {
    const double n = rint(x * 46.16624130844683);
    double r = fma(-n, 0.02166084939249829, x);
    r = fma(-n, 7.247021293269686e-19, r) + xl;
    const int ni = (int)n;
    double p = fma(r, 1.0 / 720.0, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p * r, r, r);
    const double2 t = tab[ni & 31];
    *k = ni >> 5;
    return make_double2(t.x, fma(t.x, p, t.y));
}
__device__ __forceinline__ double col_exp(double x, double xl, const double2* tab) {
    int k;
    const double2 v = col_exp2(x, xl, tab, &k);
    return ldexp(v.x + v.y, k);
}
// exp(-k u^2) as a high and a low part (to about 2^-67): the constants that
// carry a walk from run to run are the same for every column, so their errors
// do not average out, and they grow with the square of the runs walked.
__device__ __forceinline__ double2 col_exp_ku2(double k, double u, const double2* tab) {
#pragma clang fp contract(off)
    const double uh = u * u, ul = fma(u, u, -uh), a = k * uh;
    const double x = -a, xl = -(fma(k, uh, -a) + k * ul);
    const double n = rint(x * 46.16624130844683);
    const double r = fma(-n, 0.02166084939249829, x);   // exact
    const double rl = fma(-n, 7.247021293269686e-19, xl);
    const int ni = (int)n;
    double p = fma(r, 1.0 / 5040.0, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    const double c = fma(p * r, r, fma(r, rl, rl));     // exp(r + rl) = 1 + r + c
    const double2 t = tab[ni & 31];
    const double b = t.x * r, rest = fma(t.x, r, -b) + fma(t.x, c, fma(t.y, r, t.y));
    const double s = t.x + b, lo = (b - (s - t.x)) + rest, h = s + lo;
    return make_double2(ldexp(h, ni >> 5), ldexp(lo - (h - s), ni >> 5));
}

// *l += the rounding of the returned a + b.
__device__ __forceinline__ double two_sum(double a, double b, double* l) {
#pragma clang fp contract(off)
    const double s = a + b, bb = s - a;
    *l += (a - (s - bb)) + (b - bb);
    return s;
}
// exp(-(q + ql + (y + yl)^2) / 2), ql and yl small corrections, the rounding of
// the argument (up to 69) taken along.
__device__ __forceinline__ double col_weight(double q, double ql, double y, double yl, const double2* tab) {
#pragma clang fp contract(off)
    const double yy = y * y;
    double sl = ql + fma(y, y, -yy);
    const double s = two_sum(q, yy, &sl);
    return col_exp(-0.5 * s, fma(-y, yl, -0.5 * sl), tab);
}
// Kernels far narrower than a grid step: a component beyond this has a weight of
// exactly 0 (exp(-2048)), but as an argument it could overflow the reduction of
// col_exp and the polynomials (0 times infinity).  Below COL_FAR / 4 per lag the
// components of a segment stay in col_exp's range: those kernels have a loop
// without the comparison (which took 10% of a d = 4 psi_4 call).
constexpr double COL_FAR = 64.0;

// e = exp(-(q + y^2) / 2), r = exp(-u y) and the step to the next run's e, s =
// exp(-8 u y - 32 u^2) = r^8 g8, at y = y0 + u l (ql, yl: low parts of q and y0), with
// the rounding of y: at a column's far end it would shift the column's weights
// against its components.  LOW: s from r with its low part, since its error is
// multiplied by the runs walked (not for d = 4, whose columns are short: it took
// 1% of the call and changed no error).
template <bool LOW>
__device__ __forceinline__ void col_start(double q, double ql, double u, double y0, double yl, double l,
                                          const double* g8, const double2* tab, double* e, double* r, double* s) {
#pragma clang fp contract(off)
    const double ul = u * l;
    yl += fma(u, l, -ul);
    const double y = two_sum(ul, y0, &yl);
    *e = col_weight(q, ql, y, yl, tab);
    const double ru = u * y;
    int k;
    const double2 v = col_exp2(-ru, -(fma(u, y, -ru) + u * yl), tab, &k);
    const double rh = v.x + v.y;
    *r = ldexp(rh, k);
    double p = rh, pl = LOW ? v.y - (rh - v.x) : 0.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double p2 = p * p;
        if (LOW) pl = fma(2.0 * p, pl, fma(p, p, -p2));
        p = p2;
    }
    *s = ldexp(fma(p, g8[0], fma(pl, g8[0], p * g8[1])), 8 * k);
}

// Lags with |y|^2 above this are dropped: exp(-|y|^2 / 2) below 1e-30, and for
// families whose terms carry a polynomial of degree K in y (13^K at the cut)
// below 1e-30 / 13^K, so that every dropped term is below 1e-30 of its
// Gaussian's peak for all of them.
__host__ __device__ constexpr double col_cut2(int K) { return -2.0 * LOG_REL_CUT + (K > 2 ? 5.2 * K : 0.0); }

// Largest lag along an axis where the Gaussian of variance sd2 is above the
// cut (hardware root and reciprocal, good to 1e-7: rounded up by that).
__device__ __forceinline__ int col_reach(double cut2, double sd2, double delta, int lim) {
    const double v = 1.00001 * __builtin_amdgcn_sqrt(cut2 * sd2) * __builtin_amdgcn_rcp(delta);
    return (int)fmin(fmax(floor(v) + 1.0, 0.0), (double)lim);   // fmax drops a NaN
}

// An item's Gaussian k = lane & 1 (k < NGS; with one Gaussian both lanes of a
// pair do the same) from its matrix S in walk order, by the block's first
// wavefront: every lane factors, each pair of lanes writes another table entry,
// lanes 0 and 1 the rest.  Returns the normal constant; *ok is false if S is
// not positive definite (bad: not finite).
template <int D, int NGS>
__device__ __forceinline__ double col_gauss(double (&S)[D][D], const double* delta, bool bad, double cut2,
                                            const DsDev& ds, const double2* tab, ColItem<D, NGS>* it, bool* ok,
                                            double* li) {
    const int k = NGS == 2 ? threadIdx.x & 1 : 0, t = threadIdx.x >> 1;
    double sd[D], det;
#pragma unroll
    for (int p = 0; p < D; ++p) sd[p] = S[p][p];
    *ok = col_factor<D>(S, bad, li, &det);
    const double c = two_pi_pow(D) * det;
    ColGauss<D>* g = &it->g[k];
    // (the narrowest kernels are evaluated lag by lag and read no tables)
    const double u = fmin(li[tri(D - 1, D - 1)] * delta[col_axis(D, D - 1)], 1.0);
    const double2 v =
        col_exp_ku2(t < COL_RUN ? 0.5 * (double)(t * t) : t == COL_RUN ? 8.0 : t == COL_RUN + 1 ? 32.0 : 64.0, u, tab);
    if (t < COL_RUN) g->gt[t] = v.x;
    if (t >= COL_RUN && t < COL_RUN + 3) {
        double* d = t == COL_RUN ? g->h : t == COL_RUN + 1 ? g->g8 : g->h8;
        d[0] = v.x;
        d[1] = v.y;
    }
    if (t == 0) {
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int m = 0; m < D; ++m) {
                if (m <= i) g->ld[tri(i, m)] = li[tri(i, m)] * delta[col_axis(D, m)];
                g->li[i * D + m] = m <= i ? li[tri(i, m)] : 0.0;
            }
        g->c = c;
        if (k == 0) {
            it->A = ds.alag;
#pragma unroll
            for (int p = 0; p < D; ++p)
                it->lm[p] = col_reach(cut2, *ok ? sd[p] : 1.0, delta[col_axis(D, p)], ds.reach[col_axis(D, p)]);
        }
    }
    return c;
}

// Parameters of candidate h of a criterion (h >= ncand: the constant term of
// dataset h - ncand), as scv_params / pseudo_params define them, by the block's
// first wavefront.  R: order of eta_r (criteria other than SCV).  For a
// candidate's first item the slots that the final kernel reads are stored too.
template <int D, int NGS, int R>
__device__ __forceinline__ void col_crit_setup(const ScvSetup& s, int64_t h, bool first, double cut2,
                                               const double2* tab, ColItem<D, NGS>* it) {
    const ScvBatchArgs& a = s.a;
    const bool pseudo = h >= s.ncand;
    int j = 0;
    if (pseudo) {
        j = (int)(h - s.ncand);
    } else {
        int hi = a.n_ds - 1;
        while (j < hi) {
            const int mid = (j + hi + 1) >> 1;
            if (a.off[mid] <= h)
                j = mid;
            else
                hi = mid - 1;
        }
    }
    const int k = NGS == 2 ? threadIdx.x & 1 : 0, t = threadIdx.x >> 1;
    const DsDev& ds = *a.rec[j];
    constexpr int q = D * (D + 1) / 2;
    const bool scv = a.crit == KDEFFT_CRIT_SCV, qr = a.crit == KDEFFT_CRIT_QR;
    const double gw = scv ? 2.0 : 0.0, hw = k == 0 && !qr ? 2.0 : 1.0;
    double L[D][D], delta[D];
    bool sing = false;
    double ldet = 1.0;
    int o = 0;
#pragma unroll
    for (int c = 0; c < D; ++c) {
        delta[c] = ds.delta[c];
#pragma unroll
        for (int i = c; i < D; ++i) {
            const double v = pseudo ? 0.0 : s.vechL[h * q + o];
            ++o;
            L[i][c] = v;
            sing = sing || !isfinite(v) || (i == c && v == 0.0 && !pseudo);
        }
        ldet *= fabs(L[c][c]);
    }
    // S in walk order
    double S[D][D];
#pragma unroll
    for (int pi = 0; pi < D; ++pi)
#pragma unroll
        for (int pj = 0; pj <= pi; ++pj) {
            const int i = col_axis(D, pi), c = col_axis(D, pj);
            double v = 0.0;
#pragma unroll
            for (int m = 0; m <= (i < c ? i : c); ++m) v = fma(L[i][m], L[c][m], v);
            S[pi][pj] = hw * v + gw * ds.G[i * 4 + c];
        }
    double li[q];
    bool ok;
    const double c0 = col_gauss<D, NGS>(S, delta, sing, cut2, ds, tab, it, &ok, li);
    sing = __ballot(ok) != ~0ull;
    if constexpr (R > 0 || NGS == 1) {   // the eta families
        // no grid (data that are not finite): no lag is live, and the result is NaN
        double none = 0.0;
#pragma unroll
        for (int c = 0; c < D; ++c) none += 0.0 * delta[c];
        if (t == 0) it->g[k].c = c0 + none;
    }
    const double n = ds.n;
    if (t == 0) {
        const bool exact = a.crit == KDEFFT_CRIT_LSCV_EXACT;
        const double sgn = !scv && !qr && (R & 1) ? -1.0 : 1.0;
        if (k == 1 && pseudo) it->g[k].c = 0.0;
        if (k == 1 && exact) it->g[k].c *= n / (n - 1.0);
        if (k == 0) it->sign = sgn;
        if (first && k == NGS - 1) {
            // what the final kernel reads
            double* p = s.prm_out + h * PRM;
            double f = 0.0;
            if (scv) {
                double c4 = 1.0;   // (4 pi)^{-d/2}
#pragma unroll
                for (int m = 0; m < D; ++m) c4 *= 0.28209479177387814347;
                f = c4 / (n * ldet);
            } else if (!qr) {
                // eta_r(0; H) / phi_H(0): 1, -tr Q, (tr Q)^2 + 2 tr Q^2 with Q = L^{-1} L^{-T}
                double e0 = 1.0;
                if constexpr (R > 0) {
                    double tr = 0.0, tr2 = 0.0;
#pragma unroll
                    for (int x = 0; x < D; ++x)
#pragma unroll
                        for (int y = 0; y < D; ++y) {
                            double v = 0.0;
#pragma unroll
                            for (int m = 0; m <= (x < y ? x : y); ++m) v = fma(li[tri(x, m)], li[tri(y, m)], v);
                            if (x == y) tr += v;
                            tr2 = fma(v, v, tr2);
                        }
                    e0 = R == 1 ? -tr : fma(tr, tr, 2.0 * tr2);
                }
                f = sgn * (exact ? 2.0 / (n - 1.0) : 2.0 / n) * c0 * e0;
            }
            p[S_SCALE] = 1.0 / (n * n * a.prodP);
            p[S_FIRST] = pseudo ? 0.0 : f;
            p[S_SING] = sing ? 1.0 : 0.0;
            p[S_PSEUDO] = !pseudo && s.npseudo > 0 ? (double)(s.ncand + j) : -1.0;
            put_ptr(p + S_FIN_SCAL, ds.scal);
            if (s.status && !pseudo) s.status[h] = sing ? 1 : 0;
#pragma unroll
            for (int i = 0; i < D; ++i)
#pragma unroll
                for (int c = 0; c < D; ++c) p[S_L + i * 4 + c] = c <= i ? L[i][c] : 0.0;
        }
    }
}

// Parameters of psi_r at dataset h's bandwidth; the first item stores what the
// final kernel reads (L^{-1}, the normal constant times the scale of the sums).
template <int D>
__device__ __forceinline__ void col_psi_setup(const PsiBatchArgs& a, int64_t h, bool first, double cut2,
                                              double* __restrict__ prm, const double2* tab, ColItem<D, 1>* it) {
    const DsDev& ds = *a.rec[h];
    double S[D][D], delta[D], li[D * (D + 1) / 2];
#pragma unroll
    for (int pi = 0; pi < D; ++pi) {
        delta[pi] = ds.delta[pi];
#pragma unroll
        for (int pj = 0; pj <= pi; ++pj) {
            const int x = col_axis(D, pi), y = col_axis(D, pj), i = x > y ? x : y, c = x > y ? y : x;
            S[pi][pj] = a.Gv[h][c * D - c * (c - 1) / 2 + i - c];   // vech: columns of the lower triangle
        }
    }
    bool ok;   // (the bandwidths were validated on the host)
    const double c0 = col_gauss<D, 1>(S, delta, false, cut2, ds, tab, it, &ok, li);
    if (first && threadIdx.x == 0) {
        double* p = prm + h * PRM;
        double none = 0.0;   // NaN without a grid (data that are not finite): no lag is live then
#pragma unroll
        for (int i = 0; i < D; ++i) none += 0.0 * delta[i];
        p[S_C] = (c0 + none) * (1.0 / (ds.n * ds.n * a.prodP));
#pragma unroll
        for (int i = 0; i < D; ++i)
#pragma unroll
            for (int m = 0; m < D; ++m)   // L^{-1} per lag, as the walk used it
                p[S_P1 + i * D + m] = m <= i ? li[tri(i, m)] * delta[col_axis(D, m)] : 0.0;
#pragma unroll
        for (int i = 0; i < D; ++i) p[S_DELTA + i] = delta[i];
    }
}

// Exchanges within each 16 lanes (DPP): lane ^ 1, ^ 2, then the mirrored lane
// of the 8 and of the 16, so that four steps of an associative operation
// leave every lane with the result over its 16.
template <int CTRL>
__device__ __forceinline__ int dpp16(int v) { return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false); }
template <int CTRL>
__device__ __forceinline__ double dpp16(double v) {
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)dpp16<CTRL>((int)(uint32_t)b), hi = (uint32_t)dpp16<CTRL>((int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;
__device__ __forceinline__ double sum16(double v) {
    v += dpp16<DPP_XOR1>(v);
    v += dpp16<DPP_XOR2>(v);
    v += dpp16<DPP_HALF_MIRROR>(v);
    return v + dpp16<DPP_MIRROR>(v);
}
__device__ __forceinline__ int min16(int v) {
    v = min(v, dpp16<DPP_XOR1>(v));
    v = min(v, dpp16<DPP_XOR2>(v));
    v = min(v, dpp16<DPP_HALF_MIRROR>(v));
    return min(v, dpp16<DPP_MIRROR>(v));
}
__device__ __forceinline__ int max16(int v) { return -min16(-v); }

// Units of one candidate: (plane, segment of the walked axis, block of 16
// lags of the last axis), numbered with the block fastest.
template <int D>
struct ColUnits {
    int nb, nbp;       // lane blocks, of them on the positive side
    int nseg, nsn;     // segments, of them on the negative side
    int n1;            // planes along axis 1 (D = 4)
    int total;
    ColRecip<D> rnb, rnseg, rn1;
    // n0lags: lags of axis 0 the item takes (D >= 3)
    __device__ __forceinline__ ColUnits(const int* lm, int N, bool small, int n0lags) {
        const int lx = lm[D - 2], lw = lm[D - 1];
        nbp = N <= 16 ? 1 : lx / 16 + 1;
        nb = nbp + (N <= 16 ? 0 : (lx + 15) / 16);
        nsn = small ? 0 : col_side_segs(D, lw);
        nseg = small ? 1 : col_segs(D, lw);
        n1 = D == 4 ? 2 * lm[1] + 1 : 1;
        total = nb * nseg * n1 * n0lags;
        rnb = 1 / (ColRecip<D>)nb;
        rnseg = 1 / (ColRecip<D>)nseg;
        rn1 = 1 / (ColRecip<D>)n1;
    }
};

// Candidate and part of an item.  D >= 3: consecutive blocks go to the 8 dies
// in turn, so die x takes the parts x, x + 8, ... and, of each, all candidates
// one after the other: their blocks read the same planes of the lag array (at
// most about 2 MB) while those are in the die's L2.  (Candidate by candidate the
// d = 4 launch of four datasets missed the L2 on 55 of its 70 million line
// reads, 5.9 TB/s, and took 1200 us instead of 1048.)
template <int D>
__device__ __forceinline__ void col_item(const ColGeom& geo, int64_t item, int64_t nitems, int64_t* h, int* ch) {
    if (D >= 3 && (geo.nchunks & 7) == 0) {
        const uint32_t ncand = (uint32_t)(nitems / geo.nchunks), i = (uint32_t)(item >> 3), g = i / ncand;
        *ch = (int)(g * 8 + (uint32_t)(item & 7));
        *h = i - g * ncand;
    } else {
        *h = item / geo.nchunks;
        *ch = (int)(item - *h * geo.nchunks);
    }
}

// Sums of the SCV families over columns, per Gaussian: sum w and (MODE != 0)
// sum w y_a y_b.
template <int D, int MODE>
struct ColScvAcc {
    static constexpr int NGS = 2;
    static constexpr bool EXACT = false;
    static constexpr int NQ = D * (D + 1) / 2;
    static constexpr int NA = MODE == 0 ? 1 : 1 + NQ;
    double v[2][NA];
    double m[2][3];   // of the current column: sum w y_w^p
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < NA; ++i) v[k][i] = 0.0;
    }
    __device__ __forceinline__ void begin() {
#pragma unroll
        for (int k = 0; k < 2; ++k) m[k][0] = m[k][1] = m[k][2] = 0.0;
    }
    // a run of COL_RUN rows: values a, start e and ratio r, y = yE + u (t + 1)
    __device__ __forceinline__ void run(int k, const double* a, const double* g, double e, double r, double yE, double,
                                        double u) {
        double S0 = 0.0, S1 = 0.0, S2 = 0.0;
#pragma unroll
        for (int t = COL_RUN - 1; t >= 0; --t) {
            const double p = t == 0 ? a[0] : a[t] * g[t];
            S0 = t == COL_RUN - 1 ? p : fma(S0, r, p);
            if constexpr (MODE != 0) {
                S1 = t == COL_RUN - 1 ? p : fma(S1, r, S0);
                S2 = t == COL_RUN - 1 ? p : fma(S2, r, S1);
            }
        }
        S0 *= e;
        m[k][0] += S0;
        if constexpr (MODE != 0) {
            // S1 = sum s w, S2 = sum s(s+1)/2 w, s = t + 1
            const double us = u * e, b0 = yE * S0, b1 = us * S1;
            m[k][1] += b0 + b1;
            m[k][2] = fma(yE, fma(2.0, b1, b0), m[k][2]);
            m[k][2] = fma(u * us, fma(2.0, S2, -S1), m[k][2]);
        }
    }
    // one lag: weight w, walked component y (its low part not used)
    __device__ __forceinline__ void lag(int k, double w, double y, double) {
        m[k][0] += w;
        if constexpr (MODE != 0) {
            m[k][1] = fma(w, y, m[k][1]);
            m[k][2] = fma(w * y, y, m[k][2]);
        }
    }
    // the end of a column: fixed components y, column weight rw
    __device__ __forceinline__ void column(int k, double rw, const double* y) {
        const double m0 = rw * m[k][0];
        v[k][0] += m0;
        if constexpr (MODE != 0) {
            const double m1 = rw * m[k][1];
#pragma unroll
            for (int i = 0; i < D - 1; ++i) {
                const double t0 = y[i] * m0;
#pragma unroll
                for (int j = 0; j <= i; ++j) v[k][1 + tri(i, j)] = fma(t0, y[j], v[k][1 + tri(i, j)]);
                v[k][1 + tri(D - 1, i)] = fma(y[i], m1, v[k][1 + tri(D - 1, i)]);
            }
            v[k][1 + tri(D - 1, D - 1)] = fma(rw, m[k][2], v[k][1 + tri(D - 1, D - 1)]);
        }
    }
};

// Sums of the derivative families over columns, per Gaussian: with the
// whitened Hermite tensors He_alpha(y) = prod_p He_{alpha_p}(y_p),
// D^{(x)K} phi = (-1)^K (L^{-T})^{(x)K} He_K(y) phi, so the sums of order K need
// only v_alpha = sum w He_alpha, |alpha| = K: the moments He_0..He_K of the
// walked component along a column, and the products with the fixed ones' once
// per column.
template <int D, int K, int N_GS>
struct ColHermAcc {
    static constexpr int NGS = N_GS;
    // LOW: the walked components with their low parts, the polynomials to first
    // order in them (He_i' = i He_{i-1}): sums of order 4 and more cancel to 1/100 and
    // less of their terms (psi_4, M = 64, six samples: 7.7e-15 -> 6.6e-15; replayed
    // call 16.6 -> 18.2 us).
    static constexpr bool EXACT = D >= 3, LOW = D == 3 && K >= 4;
    using T = HermTab<D, K>;
    static constexpr int NA = T::NU;
    double v[NGS][NA];
    double m[NGS][K + 1];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int k = 0; k < NGS; ++k)
#pragma unroll
            for (int i = 0; i < NA; ++i) v[k][i] = 0.0;
    }
    __device__ __forceinline__ void begin() {
#pragma unroll
        for (int k = 0; k < NGS; ++k)
#pragma unroll
            for (int i = 0; i <= K; ++i) m[k][i] = 0.0;
    }
    static __device__ __forceinline__ void hermite(double y, double* he) {
        he[0] = 1.0;
        if constexpr (K > 0) he[1] = y;
#pragma unroll
        for (int i = 2; i <= K; ++i) he[i] = i == 2 ? fma(y, y, -1.0) : fma(y, he[i - 1], -(double)(i - 1) * he[i - 2]);
    }
    __device__ __forceinline__ void lag(int k, double w, double y, double yl) {
        double he[K + 1];
        hermite(y, he);
        m[k][0] += w;
#pragma unroll
        for (int i = 1; i <= K; ++i) m[k][i] = fma(w, he[i], m[k][i]);
        if constexpr (LOW) {
            const double d = w * yl;
#pragma unroll
            for (int i = 1; i <= K; ++i) m[k][i] = fma(d * i, he[i - 1], m[k][i]);
        }
    }
    __device__ __forceinline__ void run(int k, const double* a, const double* g, double e, double r, double yE, double yl,
                                        double u) {
#pragma unroll
        for (int t = 0; t < COL_RUN; ++t) {
            const double w = e * (t == 0 ? a[0] : a[t] * g[t]);
            const double y = fma(u, (double)(t + 1), yE);
            lag(k, w, y, LOW ? fma(u, (double)(t + 1), yE - y) + yl : 0.0);
            e *= r;
        }
    }
    template <int U, int... P>
    static __device__ __forceinline__ double lead(const double (*he)[K + 1], std::integer_sequence<int, P...>) {
        double x = 1.0;
        ((T::tab.a[T::NB - T::NU + U][P] > 0 ? (x *= he[P][T::tab.a[T::NB - T::NU + U][P]]) : 0.0), ...);
        return x;
    }
    template <int... U>
    __device__ __forceinline__ void add(int k, double rw, const double (*he)[K + 1], std::integer_sequence<int, U...>) {
        ((v[k][U] = fma(rw * lead<U>(he, std::make_integer_sequence<int, D - 1>{}),
                        m[k][T::tab.a[T::NB - T::NU + U][D - 1]], v[k][U])),
         ...);
    }
    __device__ __forceinline__ void column(int k, double rw, const double* y) {
        double he[D > 1 ? D - 1 : 1][K + 1];
#pragma unroll
        for (int p = 0; p < D - 1; ++p) hermite(y[p], he[p]);
        add(k, rw, he, std::make_integer_sequence<int, NA>{});
    }
};

// Grid size for nitems work items (cols.hip).
int64_t cols_blocks(int64_t nitems, int grid_blocks);

// Part ch of an item's candidate, walked into acc (see the top).  SMALL: the
// walked axis has P < 16 (at most 7 lags): one segment, rows addressed and
// masked one by one.
template <int D, bool SMALL, class Acc>
__device__ __forceinline__ void col_walk(const ColGeom& geo, int ch, const ColItem<D, Acc::NGS>& it,
                                         const double2* s_exp, double cut2, Acc& acc) {
    constexpr int NGS = Acc::NGS;
    const int tid = threadIdx.x, l16 = tid & 15;
    double uw[NGS];
    bool near1 = true, far = false;   // far: components beyond COL_FAR are possible
#pragma unroll
    for (int k = 0; k < NGS; ++k) {
        uw[k] = wave_uniform(it.g[k].ld[tri(D - 1, D - 1)]);
        near1 = near1 && uw[k] * uw[k] < 0.69314718055994531;
        far = far || uw[k] > COL_FAR / 4;
    }
    // (a pointer taken from memory: named global so that its loads are not flat ones)
    using gptr = const __attribute__((address_space(1))) char*;
    const gptr A = reinterpret_cast<gptr>(static_cast<uintptr_t>(
        __double_as_longlong(wave_uniform(__longlong_as_double((long long)(uintptr_t)it.A)))));
    using gdbl = const __attribute__((address_space(1))) double*;
    int lm[D];
#pragma unroll
    for (int p = 0; p < D; ++p) lm[p] = __builtin_amdgcn_readfirstlane(it.lm[p]);

    if constexpr (D == 1) {
        // one lag per lane, the mirror lag counted by weight 2
        acc.begin();
        for (int l = ch * COL_NT + tid; l <= lm[0]; l += (int)geo.nchunks * COL_NT) {
            const double a = (l == 0 ? 1.0 : 2.0) * *reinterpret_cast<gdbl>(A + (size_t)l * 8);
#pragma unroll
            for (int k = 0; k < NGS; ++k) {
                const double y = uw[k] * (double)l;
                if (fabs(y) < COL_FAR) acc.lag(k, exp(-0.5 * y * y) * a, y, 0.0);
            }
        }
#pragma unroll
        for (int k = 0; k < NGS; ++k) acc.column(k, 1.0, nullptr);
    } else {
        constexpr int SEG = COL_SEG;
        const int N = geo.P[D - 1], Pw = geo.P[D - 2];
        // D >= 3: part ch takes the lags c0, 2 n0 - 1 - c0, 2 n0 + c0, ... of
        // axis 0 (c0 = ch mod n0) and every nsub-th block step of their units;
        // D = 2: every nchunks-th block step
        const int n0 = D >= 3 ? geo.n0 : 1, c0 = D >= 3 ? ch % n0 : 0;
        const int sub = D >= 3 ? ch / n0 : ch, nsub = (int)geo.nchunks / n0;
        auto lag0 = [&](int j) { return j & 1 ? (j + 1) * n0 - 1 - c0 : j * n0 + c0; };
        const int j0 = lm[0] / n0;
        const ColUnits<D> un(lm, N, SMALL, D >= 3 ? j0 + (lag0(j0) <= lm[0] ? 1 : 0) : 1);
        const double iu = 1.0 / uw[0];
        double g[NGS][COL_RUN], hh[NGS][2], h8[NGS][2];
#pragma unroll
        for (int k = 0; k < NGS; ++k) {
#pragma unroll
            for (int t = 1; t < COL_RUN; ++t) g[k][t] = wave_uniform(it.g[k].gt[t]);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                hh[k][i] = wave_uniform(it.g[k].h[i]);
                h8[k][i] = wave_uniform(it.g[k].h8[i]);
            }
        }
        const uint32_t strideP = (uint32_t)Pw * (uint32_t)N;   // elements of a plane
        for (int u = sub * 16 + (tid >> 4); u < un.total; u += nsub * 16) {
            // decode: block fastest, then segment, then plane
            const int rs = col_quot(u, un.rnb);
            const int b = u - rs * un.nb;
            const int pl = col_quot(rs, un.rnseg);
            const int seg = rs - pl * un.nseg;
            int lag[D];
            double rw = 2.0;
            uint32_t col = 0;   // element offset of the column in the half set (below 2^29: prod P <= 2^30)
            if constexpr (D == 3) {
                lag[0] = lag0(pl);
                col += (uint32_t)lag[0] * strideP;
            }
            if constexpr (D == 4) {
                const int i0 = col_quot(pl, un.rn1);
                const int l1 = pl - i0 * un.n1 - lm[1];
                lag[0] = lag0(i0);
                lag[1] = l1;
                col += ((uint32_t)lag[0] * (uint32_t)geo.P[1] + (uint32_t)(l1 & (geo.P[1] - 1))) * strideP;
            }
            if constexpr (D >= 3) rw = lag[0] == 0 ? 1.0 : 2.0;
            const int idx = (b < un.nbp ? b * 16 : N - 16 * (b - un.nbp + 1)) + l16;
            const bool inrow = idx < N;
            lag[D - 2] = idx < N / 2 ? idx : idx - N;
            col += inrow ? idx : 0;
            const int wl = lm[D - 1];
            const int s0 = SMALL ? (D >= 3 ? -wl : 0) : (seg - un.nsn) * SEG - (D == 2 ? 0 : SEG / 2);
            // whitened fixed components (and, last, the walked one at lag 0)
            auto whiten = [&](int k, double* y) {
#pragma unroll
                for (int p = 0; p < D; ++p) {
                    double v = 0.0;
#pragma unroll
                    for (int j = 0; j <= (p < D - 1 ? p : D - 2); ++j) v = fma(it.g[k].ld[tri(p, j)], (double)lag[j], v);
                    y[p] = v;
                }
            };
            // the same, rounded once, and its low part
            auto whiten_exact = [&](int k, double* y, double* l) {
#pragma unroll
                for (int p = 0; p < D; ++p) {
                    double v = 0.0, w = 0.0;
#pragma unroll
                    for (int j = 0; j <= (p < D - 1 ? p : D - 2); ++j) {
                        const double c = it.g[k].ld[tri(p, j)], x = (double)lag[j], cx = c * x;
                        w += fma(c, x, -cx);
                        v = two_sum(v, cx, &w);
                    }
                    y[p] = v + w;
                    l[p] = w - (y[p] - v);
                }
            };
            // Few columns carry a narrow kernel's sums, and sums of high order cancel,
            // so that a component's or the exponent's rounding would not average out:
            // there both are kept with their low parts.  (psi_4, d = 4, M = 32, mean
            // error of the largest entry over ten samples against extended precision
            // 9.7e-15; a row walk with S^{-1} 9.9e-15.)
            double yE[NGS], yl[NGS], q[NGS], ql[NGS];   // yE: the walked component at lag 0
            auto exact = [&](int k) {
                double y[D], l[D];
                whiten_exact(k, y, l);
                q[k] = ql[k] = 0.0;
#pragma unroll
                for (int p = 0; p < D - 1; ++p) {
                    const double yy = y[p] * y[p];
                    ql[k] += fma(2.0 * y[p], l[p], fma(y[p], y[p], -yy));
                    q[k] = two_sum(q[k], yy, &ql[k]);
                }
                yE[k] = y[D - 1];
                yl[k] = l[D - 1];
            };
#pragma unroll
            for (int k = 0; k < NGS; ++k) {
                if constexpr (Acc::EXACT) {
                    exact(k);
                } else {
                    double y[D];
                    whiten(k, y);
                    q[k] = 0.0;
#pragma unroll
                    for (int p = 0; p < D - 1; ++p) q[k] = fma(y[p], y[p], q[k]);
                    yE[k] = y[D - 1];
                    ql[k] = yl[k] = 0.0;
                }
            }
            // live rows of this column, as runs of the segment
            int ca = 127, cb = -1;
            if (inrow && q[0] <= cut2) {
                const double hw = sqrt(cut2 - q[0]) * iu, ctr = -yE[0] * iu;
                const double lo = s0 > -wl ? s0 : -wl;
                const double hi = SMALL || s0 + SEG - 1 > wl ? wl : s0 + SEG - 1;
                const double fa = fmax(floor(ctr - hw), lo), fb = fmin(ceil(ctr + hw), hi);
                if (fa <= fb) {
                    ca = ((int)fa - s0) / COL_RUN;
                    cb = ((int)fb - s0) / COL_RUN;
                }
            }
            const int ga = min16(ca), gb = max16(cb);
            if (gb < 0) continue;
            // uniform base, 32-bit byte offset per lane
            auto at = [&](int l, int t) {
                const uint32_t off = (col + (uint32_t)(l & (Pw - 1)) * (uint32_t)N) * 8u;
                return *reinterpret_cast<gdbl>(A + (size_t)t * N * 8 + off);
            };
            auto fetch = [&](int c, double* av) {
                const int l = s0 + COL_RUN * c;
#pragma unroll
                for (int t = 0; t < COL_RUN; ++t) {
                    if constexpr (SMALL)
                        av[t] = l + t <= wl ? at(l + t, 0) : 0.0;
                    else
                        av[t] = at(l, t);
                }
                if (D == 2 && l == 0) av[0] *= 0.5;   // row 0 is its own mirror
            };
            acc.begin();
            if (near1) {
                double e[NGS], r[NGS], st[NGS];
                const double ls = (double)(s0 + COL_RUN * (cb >= 0 ? ca : 0));
#pragma unroll
                for (int k = 0; k < NGS; ++k)
                    col_start<(D < 4)>(q[k], ql[k], uw[k], yE[k], yl[k], ls, it.g[k].g8, s_exp, &e[k], &r[k], &st[k]);
                auto run = [&](int c, const double* av) {
                    if (c < ca) return;   // the lane's column starts in a later run
                    const double before = (double)(s0 + COL_RUN * c - 1);
#pragma unroll
                    for (int k = 0; k < NGS; ++k) {
                        const double yb = fma(uw[k], before, yE[k]);
                        acc.run(k, av, g[k], e[k], r[k], yb, fma(uw[k], before, yE[k] - yb) + yl[k], uw[k]);
                        e[k] *= st[k];
                        // (exact products with the high parts)
                        st[k] = fma(st[k], h8[k][0], st[k] * h8[k][1]);
                        r[k] = fma(r[k], hh[k][0], r[k] * hh[k][1]);
                    }
                };
                double a0[COL_RUN], a1[COL_RUN];   // the next run's loads are in flight over the current one
                fetch(ga, a0);
                for (int c = ga; c <= gb; c += 2) {
                    fetch(c < gb ? c + 1 : gb, a1);
                    run(c, a0);
                    if (c >= gb) break;
                    fetch(c + 1 < gb ? c + 2 : gb, a0);
                    run(c + 1, a1);
                }
            } else if (cb >= 0) {
                // narrow kernels: lag by lag
                if constexpr (!Acc::EXACT) {
#pragma unroll
                    for (int k = 0; k < NGS; ++k) exact(k);
                }
                auto lags = [&](auto guarded) {
#pragma unroll 1
                    for (int l = s0 + COL_RUN * ga; l < s0 + COL_RUN * (gb + 1); ++l) {
                        double a = 0.0;
                        if (!SMALL || l <= wl) a = at(l, 0);
                        if (D == 2 && l == 0) a *= 0.5;
#pragma unroll
                        for (int k = 0; k < NGS; ++k) {
                            const double ul = uw[k] * (double)l;
                            double low = yl[k] + fma(uw[k], (double)l, -ul);
                            const double yw = two_sum(ul, yE[k], &low);
                            if (guarded && fabs(yw) >= COL_FAR) continue;
                            acc.lag(k, col_weight(q[k], ql[k], yw, low, s_exp) * a, yw, low);
                        }
                    }
                };
                if (far)
                    lags(std::true_type{});
                else
                    lags(std::false_type{});
            }
            // the column's sums: products with the fixed components (formed
            // again: kept over the walk they would cost registers)
#pragma unroll
            for (int p = 0; p < D - 1; ++p) asm volatile("" : "+v"(lag[p]));
#pragma unroll
            for (int k = 0; k < NGS; ++k) {
                double y[D], l[D];
                if (near1 && !Acc::EXACT)
                    whiten(k, y);
                else
                    whiten_exact(k, y, l);
                acc.column(k, rw, y);
            }
        }
    }
}

// Block sums of the accumulators, fixed order, into s_tot [NGS * NA].
template <class Acc>
__device__ __forceinline__ void col_reduce(const Acc& acc, double (*s_red)[Acc::NGS * Acc::NA], double* s_tot) {
    constexpr int NV = Acc::NGS * Acc::NA;
    const int tid = threadIdx.x;
#pragma unroll
    for (int k = 0; k < Acc::NGS; ++k)
#pragma unroll
        for (int i = 0; i < Acc::NA; ++i) {
            const double v = sum16(acc.v[k][i]);
            if ((tid & 15) == 0) s_red[tid >> 4][k * Acc::NA + i] = v;
        }
    __syncthreads();
    if (tid < NV) {
        double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int w = 0; w < COL_NT / 16; ++w) v[w & 3] += s_red[w][tid];
        s_tot[tid] = (v[0] + v[1]) + (v[2] + v[3]);
    }
    __syncthreads();
}

// The SCV families: ScvFun's modes (0 objective, 1 objective and gradient,
// 2 gradient).
template <int D, int MODE, bool SMALL>
__global__ __launch_bounds__(COL_NT, D <= 2 ? 4 : 3) void k_cols_scv(ColGeom geo, ScvSetup setup, int64_t nitems,
                                                                     double* __restrict__ partial) {
    using Acc = ColScvAcc<D, MODE>;
    constexpr int NG = ScvFun<D, MODE>::NG, NA = Acc::NA;
    constexpr double cut2 = col_cut2(2);
    __shared__ ColItem<D, 2> s_it;
    __shared__ double s_red[COL_NT / 16][2 * NA], s_tot[2 * NA];
    __shared__ double2 s_exp[32];
    const int tid = threadIdx.x;
    if (tid < 32) s_exp[tid] = COL_EXP2[tid];   // (the first wavefront's own, for the set-up)
    for (int64_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        int64_t h;
        int ch;
        col_item<D>(geo, item, nitems, &h, &ch);
        if (tid < 64) col_crit_setup<D, 2, 0>(setup, h, ch == 0, cut2, s_exp, &s_it);
        __syncthreads();
        Acc acc;
        acc.clear();
        col_walk<D, SMALL>(geo, ch, s_it, s_exp, cut2, acc);
        col_reduce(acc, s_red, s_tot);
        // the outputs: c_k times the sums, the second-order ones transformed
        // back by L^{-1}
        if (tid < NG) {
            double out;
            if (MODE != 2 && tid == 0) {
                out = s_it.g[0].c * s_tot[0] - 2.0 * s_it.g[1].c * s_tot[NA];
            } else {
                // output number tid: D_ij, i <= j in axis order, at its walk positions
                int pi = 0, pj = 0, o = MODE == 2 ? 0 : 1;
#pragma unroll
                for (int i = 0; i < D; ++i)
#pragma unroll
                    for (int j = i; j < D; ++j, ++o)
                        if (tid == o) {
                            pi = col_pos(D, i);
                            pj = col_pos(D, j);
                        }
                double hs[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const double* li = s_it.g[k].li;
                    double v = 0.0;
#pragma unroll
                    for (int a = 0; a < D; ++a) {
                        double r = 0.0;
#pragma unroll
                        for (int b = 0; b < D; ++b) {
                            const int ab = MODE == 0 ? 0 : 1 + (a >= b ? tri(a, b) : tri(b, a));
                            r = fma(s_tot[k * NA + ab] - (a == b ? s_tot[k * NA] : 0.0), li[b * D + pj], r);
                        }
                        v = fma(li[a * D + pi], r, v);
                    }
                    hs[k] = s_it.g[k].c * v;
                }
                out = hs[0] - hs[1];
            }
            partial[(h * geo.nchunks + ch) * NG + tid] = out;
        }
        __syncthreads();
    }
}

template <int D, int R>
constexpr int col_psi_occ() { return HermTab<D, R>::NU > 20 ? 2 : 3; }

// psi_r: partial sums of the whitened tensor's unique entries (walk order);
// k_cols_psi_final adds and transforms them.
template <int D, int R, bool SMALL>
__global__ __launch_bounds__(COL_NT, (col_psi_occ<D, R>())) void k_cols_psi(ColGeom geo, PsiBatchArgs args, int64_t nitems,
                                                                           double* __restrict__ prm,
                                                                           double* __restrict__ partial) {
    using Acc = ColHermAcc<D, R, 1>;
    constexpr int NA = Acc::NA;
    constexpr double cut2 = col_cut2(R);
    __shared__ ColItem<D, 1> s_it;
    __shared__ double s_red[COL_NT / 16][NA], s_tot[NA];
    __shared__ double2 s_exp[32];
    const int tid = threadIdx.x;
    if (tid < 32) s_exp[tid] = COL_EXP2[tid];
    for (int64_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        int64_t h;
        int ch;
        col_item<D>(geo, item, nitems, &h, &ch);
        if (tid < 64) col_psi_setup<D>(args, h, ch == 0, cut2, prm, s_exp, &s_it);
        __syncthreads();
        Acc acc;
        acc.clear();
        col_walk<D, SMALL>(geo, ch, s_it, s_exp, cut2, acc);
        col_reduce(acc, s_red, s_tot);
        if (tid < NA) partial[(h * geo.nchunks + ch) * NA + tid] = s_tot[tid];
        __syncthreads();
    }
}

__host__ __device__ constexpr int ipow(int b, int e) { return e == 0 ? 1 : b * ipow(b, e - 1); }

// Index of the unique entry (walk order) of the full tensor's element e.
template <int D, int R>
struct ColTensor {
    static constexpr int NF = ipow(D, R);
    struct Tab {
        unsigned char u[NF];
    };
    static constexpr Tab make() {
        using T = HermTab<D, R>;
        Tab t{};
        for (int e = 0; e < NF; ++e) {
            int cnt[4] = {0, 0, 0, 0}, x = e;
            for (int m = 0; m < R; ++m) {
                cnt[x % D] += 1;
                x /= D;
            }
            for (int b = 0; b < T::NU; ++b) {
                bool eq = true;
                for (int p = 0; p < D; ++p) eq = eq && T::tab.a[T::NB - T::NU + b][p] == cnt[p];
                if (eq) t.u[e] = (unsigned char)b;
            }
        }
        return t;
    }
    static constexpr Tab tab = make();
};
template <int D, int R>
static __device__ const typename ColTensor<D, R>::Tab COL_TENSOR = ColTensor<D, R>::make();
// The full tensor's element of each unique entry (axis order, sorted tuples).
template <int D, int R>
struct ColUnique {
    struct Tab {
        short e[HermTab<D, R>::NU];
    };
    static constexpr Tab make() {
        using T = HermTab<D, R>;
        Tab t{};
        for (int b = 0; b < T::NU; ++b) {
            int e = 0;
            for (int k = 0; k < D; ++k)
                for (int m = 0; m < T::tab.a[T::NB - T::NU + b][k]; ++m) e = e * D + k;
            t.e[b] = (short)e;
        }
        return t;
    }
};
template <int D, int R>
static __device__ const typename ColUnique<D, R>::Tab COL_UNIQUE = ColUnique<D, R>::make();

// psi_r of dataset blockIdx.x: the parts' sums added in a fixed order, then the
// tensor transformed by L^{-1} mode by mode.
template <int D, int R>
__global__ __launch_bounds__(COL_NT) void k_cols_psi_final(const double* __restrict__ partial, int64_t nchunks,
                                                           const double* __restrict__ prm, double* __restrict__ psi) {
    constexpr int NU = HermTab<D, R>::NU, NF = ipow(D, R), NR = COL_NT / NU;
    __shared__ double s_part[NR * NU], s_t[2][NF], s_li[D * D], s_dl[D];
    const int tid = threadIdx.x;
    const int64_t h = blockIdx.x;
    if (tid < D * D) s_li[tid] = prm[h * PRM + S_P1 + tid];
    if (tid < D) s_dl[tid] = prm[h * PRM + S_DELTA + tid];
    const double scale = prm[h * PRM + S_C];
    if (tid < NR * NU) {
        const double* p = partial + h * nchunks * NU;
        const int n = (int)nchunks * NU;
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        int e = tid;
        for (; e + 3 * NR * NU < n; e += 4 * NR * NU) {   // (four loads in flight)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] += p[e + i * NR * NU];
        }
        for (; e < n; e += NR * NU) s[0] += p[e];
        s_part[tid] = (s[0] + s[1]) + (s[2] + s[3]);
    }
    __syncthreads();
    for (int e = tid; e < NU; e += COL_NT) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int r = 0; r < NR; ++r) s[r & 3] += s_part[r * NU + e];
        s_t[1][e] = (s[0] + s[1]) + (s[2] + s[3]);   // (unique entries; NU <= NF)
    }
    __syncthreads();
    for (int e = tid; e < NF; e += COL_NT) s_t[0][e] = s_t[1][R > 0 ? COL_TENSOR<D, R>.u[e] : 0];
    __syncthreads();
    // each mode: positions (rows of L^{-1}) to axes
    int cur = 0;
    int st = 1;
#pragma unroll
    for (int m = 0; m < R; ++m, st *= D) {   // (unrolled: divisions by constants)
        for (int e = tid; e < NF; e += COL_NT) {
            const int i = (e / st) % D, base = e - i * st;
            const int pi = D == 1 ? 0 : (i < D - 2 ? i : (i == D - 2 ? D - 1 : D - 2));   // position of axis i
            double s = 0.0;
#pragma unroll
            for (int p = 0; p < D; ++p) s = fma(s_t[cur][base + p * st], s_li[p * D + pi], s);
            s_t[cur ^ 1][e] = s;
        }
        __syncthreads();
        cur ^= 1;
    }
    for (int e = tid; e < NU; e += COL_NT) {
        int x = R > 0 ? COL_UNIQUE<D, R>.e[e] : 0;
        double v = scale * s_t[cur][x];
#pragma unroll
        for (int m = 0; m < R; ++m, x /= D) v /= s_dl[x % D];   // from lags to the axes' units
        psi[h * NU + e] = v;
    }
}

// Scalar eta_r families (Q_r with one Gaussian, LSCV_r with two), r <= 2:
// eta_r = (tr of the tensor pairs) = sum over pairs Q_{ab} .. He_{2r}, with
// Q = L^{-1} L^{-T} in whitened coordinates.
template <int D, int NGS, int R, bool SMALL>
__global__ __launch_bounds__(COL_NT, 3) void k_cols_eta(ColGeom geo, ScvSetup setup, int64_t nitems,
                                                        double* __restrict__ partial) {
    constexpr int K = 2 * R, NF = ipow(D, K);
    using Acc = ColHermAcc<D, K, NGS>;
    constexpr int NA = Acc::NA;
    constexpr double cut2 = col_cut2(K);
    __shared__ ColItem<D, NGS> s_it;
    __shared__ double s_red[COL_NT / 16][NGS * NA], s_tot[NGS * NA], s_q[NGS][D * D], s_w[COL_NT / 16];
    __shared__ double2 s_exp[32];
    const int tid = threadIdx.x;
    if (tid < 32) s_exp[tid] = COL_EXP2[tid];
    for (int64_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        int64_t h;
        int ch;
        col_item<D>(geo, item, nitems, &h, &ch);
        if (tid < 64) col_crit_setup<D, NGS, R>(setup, h, ch == 0, cut2, s_exp, &s_it);
        __syncthreads();
        if (tid < NGS * D * D) {
            const int k = tid / (D * D), a = (tid / D) % D, b = tid % D;
            double v = 0.0;
#pragma unroll
            for (int m = 0; m < D; ++m) v = fma(s_it.g[k].li[a * D + m], s_it.g[k].li[b * D + m], v);
            s_q[k][a * D + b] = v;
        }
        Acc acc;
        acc.clear();
        col_walk<D, SMALL>(geo, ch, s_it, s_exp, cut2, acc);
        col_reduce(acc, s_red, s_tot);
        // contraction: one element of the full tensor per thread
        static_assert(NGS * NF <= COL_NT, "one element per thread");
        double v = 0.0;
        if (tid < NGS * NF) {
            const int k = tid / NF, e = tid % NF;
            v = (k == 0 ? 1.0 : -2.0) * s_it.g[k].c;
            if constexpr (R == 0) v *= s_tot[k * NA];
            if constexpr (R == 1) v *= s_q[k][e] * s_tot[k * NA + COL_TENSOR<D, K>.u[e]];
            if constexpr (R == 2) v *= s_q[k][e % (D * D)] * s_q[k][e / (D * D)] * s_tot[k * NA + COL_TENSOR<D, K>.u[e]];
        }
        v = sum16(v);
        if ((tid & 15) == 0) s_w[tid >> 4] = v;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < COL_NT / 16; ++w) s += s_w[w];
            partial[h * geo.nchunks + ch] = s_it.sign * s;
        }
        __syncthreads();
    }
}

}  // namespace kdefft
