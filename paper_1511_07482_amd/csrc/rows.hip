// Host dispatch of the batched row kernels, and the small per-candidate
// kernels around them: SCV parameter setup (Cholesky factors of 2H+2G and
// H+2G) and the final assembly of psi / SCV objective / gradient from the
// per-item partial sums (fixed summation order).
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "dev_kernels.h"
#include "eta_fun.h"
#include "finish.h"
#include "minstep.h"
#include "internal.h"
#include "params.h"
#include "rows_impl.h"

namespace kdefft {

hipError_t launch_rows_d1(int, int, int, int, const double*, RowGeom, int64_t, double*, int, const double2*,
                          hipStream_t);
hipError_t launch_rows_d2(int, int, int, int, const double*, RowGeom, int64_t, double*, int, const double2*,
                          hipStream_t);
hipError_t launch_rows_d3(int, int, int, int, const double*, RowGeom, int64_t, double*, int, const double2*,
                          hipStream_t);
hipError_t launch_rows_d4(int, int, int, int, const double*, RowGeom, int64_t, double*, int, const double2*,
                          hipStream_t);
hipError_t launch_rows_eta_d1(int, int, int, int, const double*, RowGeom, int64_t, double*, int, hipStream_t);
hipError_t launch_rows_eta_d2(int, int, int, int, const double*, RowGeom, int64_t, double*, int, hipStream_t);
hipError_t launch_rows_eta_d3(int, int, int, int, const double*, RowGeom, int64_t, double*, int, hipStream_t);
hipError_t launch_rows_eta_d4(int, int, int, int, const double*, RowGeom, int64_t, double*, int, hipStream_t);
int rows_iter_eta_d1(int, int, int);
int rows_iter_eta_d2(int, int, int);
int rows_iter_eta_d3(int, int, int);
int rows_iter_eta_d4(int, int, int);
int rows_iter_d1(int, int, int, int);
int rows_iter_d2(int, int, int, int);
int rows_iter_d3(int, int, int, int);
int rows_iter_d4(int, int, int, int);

static int binom_h(int n, int k) {
    int r = 1;
    for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
    return r;
}

template <int N>
static int layout_of(int moments, int* run_len, int* runs_per_seg, int* rows_per_pass) {
    if (moments) {
        constexpr int RL = mom_run_of<N>() < N / 2 ? mom_run_of<N>() : N / 2;
        *run_len = RL;
        *runs_per_seg = mom_seg_of<N, RL>();
        *rows_per_pass = mom_rows_per_pass<N>();
    } else {
        *run_len = LAG_RUN;
        *runs_per_seg = 1;
        *rows_per_pass = lag_rows_per_pass<N>();
    }
    return 1;
}

int lag_layout(int N, int moments, int* run_len, int* runs_per_seg, int* rows_per_pass) {
    switch (N) {
        case 4: return layout_of<4>(moments, run_len, runs_per_seg, rows_per_pass);
        case 8: return layout_of<8>(moments, run_len, runs_per_seg, rows_per_pass);
        case 16: return layout_of<16>(moments, run_len, runs_per_seg, rows_per_pass);
        case 32: return layout_of<32>(moments, run_len, runs_per_seg, rows_per_pass);
        case 64: return layout_of<64>(moments, run_len, runs_per_seg, rows_per_pass);
        case 128: return layout_of<128>(moments, run_len, runs_per_seg, rows_per_pass);
        case 256: return layout_of<256>(moments, run_len, runs_per_seg, rows_per_pass);
        case 512: return layout_of<512>(moments, run_len, runs_per_seg, rows_per_pass);
        case 1024: return layout_of<1024>(moments, run_len, runs_per_seg, rows_per_pass);
        case 2048: return layout_of<2048>(moments, run_len, runs_per_seg, rows_per_pass);
        default: return 0;
    }
}

int ng_of(int kind, int d, int r) {
    const int q = d * (d + 1) / 2;
    switch (kind) {
        case FUN_PSI: return binom_h(d + r - 1, r);
        case FUN_SCV_OBJ: return 1;
        case FUN_SCV_OBJGRAD: return 1 + q;
        case FUN_SCV_GRAD: return q;
        case FUN_ETA1:
        case FUN_ETA2: return 1;
        default: return 0;
    }
}

int rows_per_iter(int kind, int d, int r, int N, int variant) {
    if (kind == FUN_ETA1 || kind == FUN_ETA2) {
        switch (d) {
            case 1: return rows_iter_eta_d1(kind, N, variant);
            case 2: return rows_iter_eta_d2(kind, N, variant);
            case 3: return rows_iter_eta_d3(kind, N, variant);
            case 4: return rows_iter_eta_d4(kind, N, variant);
            default: return 0;
        }
    }
    switch (d) {
        case 1: return rows_iter_d1(kind, r, N, variant);
        case 2: return rows_iter_d2(kind, r, N, variant);
        case 3: return rows_iter_d3(kind, r, N, variant);
        case 4: return rows_iter_d4(kind, r, N, variant);
        default: return 0;
    }
}

RowGeom make_geom(const kdefft_grid& g, int kind, int r, int64_t ncand, int variant, int64_t max_chunks) {
    RowGeom geo{};
    geo.d = g.d;
    for (int k = 0; k < 4; ++k) {
        geo.M[k] = k < g.d ? g.M[k] : 1;
        geo.P[k] = k < g.d ? g.P[k] : 1;
    }
    int64_t nrows = 1;
    if (g.d >= 2) {
        nrows = g.M[0];
        for (int k = 1; k + 1 < g.d; ++k) nrows *= (2 * g.M[k] - 1);
    }
    geo.nrows = nrows;
    geo.Q = g.P[g.d - 1] / 2 + 1;
    int ri = rows_per_iter(kind, g.d, r, g.P[g.d - 1], variant);
    if (ri < 1) ri = 1;
    // lag kernel: larger items amortise the per-item set-up and block reduction
    const int64_t target = variant >= 3 ? 2048 : 8192;
    int64_t iters = (nrows * ncand + (int64_t)ri * target - 1) / ((int64_t)ri * target);
    if (iters < 1) iters = 1;
    int64_t chunk = iters * ri;
    if (max_chunks < 1) max_chunks = 1;
    // (items of at least nrows / max_chunks rows; not from nrows + max_chunks - 1, which may overflow)
    const int64_t least = nrows / max_chunks + (nrows % max_chunks ? 1 : 0);
    if (chunk < least) chunk = (least + ri - 1) / ri * ri;
    if (chunk > nrows) chunk = ((nrows + ri - 1) / ri) * ri;
    geo.chunk = chunk;
    geo.nchunks = (nrows + chunk - 1) / chunk;
    return geo;
}

hipError_t launch_rows(int kind, int d, int r, const RowGeom& geo, const double* prm, int64_t ncand,
                       double* partial, const RowLaunch& rl, hipStream_t s) {
    // only the spectral variants read the twiddle table (set up on first use)
    const double2* tw = nullptr;
    if (rl.variant < 3 && kind != FUN_ETA1 && kind != FUN_ETA2) {
        hipError_t e = twiddles(&tw);
        if (e != hipSuccess) return e;
    }
    const int64_t nitems = ncand * geo.nchunks;
    const int N = geo.P[d - 1];
    if (kind == FUN_ETA1 || kind == FUN_ETA2) {
        switch (d) {
            case 1: return launch_rows_eta_d1(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, s);
            case 2: return launch_rows_eta_d2(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, s);
            case 3: return launch_rows_eta_d3(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, s);
            case 4: return launch_rows_eta_d4(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, s);
            default: return hipErrorInvalidValue;
        }
    }
    switch (d) {
        case 1: return launch_rows_d1(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, tw, s);
        case 2: return launch_rows_d2(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, tw, s);
        case 3: return launch_rows_d3(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, tw, s);
        case 4: return launch_rows_d4(kind, r, N, rl.variant, prm, geo, nitems, partial, rl.grid_blocks, tw, s);
        default: return hipErrorInvalidValue;
    }
}

// One wavefront per candidate (real ones, then npseudo constant-term
// candidates): lane 0 writes the parameter block; with wc set, the wavefront
// then counts the candidate's live runs of rl lags over all rows of the half
// lag set (row_live) into wc[c].
template <int D>
__global__ __launch_bounds__(256) void k_scv_setup(const double* __restrict__ vechL, ScvBatchArgs a, int64_t ncand,
                                                   int npseudo, double* __restrict__ prm,
                                                   int32_t* __restrict__ status, RowGeom geo, int rl,
                                                   int32_t* __restrict__ wc) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * 4 + wave;
    const bool active = c < ncand + npseudo;
    if (active && lane == 0) {
        if (c < ncand)
            scv_params<D>(vechL, a, c, ncand, npseudo, prm + c * PRM, status);
        else
            pseudo_params<D>(a, (int)(c - ncand), prm + c * PRM);
    }
    if (!wc) return;   // grid-uniform
    __syncthreads();   // the blocks written by lane 0 are visible to the block
    if (!active) return;
    const double* p = prm + c * PRM;
    ScvFun<D, 1> f;
    f.load(p);
    double delta[D];
#pragma unroll
    for (int k = 0; k < D; ++k) delta[k] = p[S_DELTA + k];
    const int M_last = geo.M[D - 1], N = geo.P[D - 1];
    int units = 0;
    for (int64_t row = lane; row < geo.nrows; row += 64) {
        const LiveRuns lr = row_live<D>(f, row_info<D>(row, geo.nrows, geo, delta, nullptr), M_last, N, rl, delta[D - 1]);
        units += lr.pn + lr.nn;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) units += __shfl_xor(units, off, 64);
    if (lane == 0) wc[c] = units;
}

hipError_t launch_scv_setup(const double* vechL, const ScvBatchArgs& a, int64_t ncand, int npseudo, double* prm,
                            int32_t* status, const RowGeom& geo, int32_t* wc, hipStream_t s) {
    const int64_t blocks = (ncand + npseudo + 3) / 4;
    int rl = 1, seg = 1, rows = 1;
    if (wc && !lag_layout(geo.P[geo.d - 1], 1, &rl, &seg, &rows)) return hipErrorInvalidValue;
    switch (a.d) {
        case 1: hipLaunchKernelGGL(k_scv_setup<1>, dim3((unsigned)blocks), dim3(256), 0, s, vechL, a, ncand, npseudo, prm, status, geo, rl, wc); break;
        case 2: hipLaunchKernelGGL(k_scv_setup<2>, dim3((unsigned)blocks), dim3(256), 0, s, vechL, a, ncand, npseudo, prm, status, geo, rl, wc); break;
        case 3: hipLaunchKernelGGL(k_scv_setup<3>, dim3((unsigned)blocks), dim3(256), 0, s, vechL, a, ncand, npseudo, prm, status, geo, rl, wc); break;
        case 4: hipLaunchKernelGGL(k_scv_setup<4>, dim3((unsigned)blocks), dim3(256), 0, s, vechL, a, ncand, npseudo, prm, status, geo, rl, wc); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// One thread per dataset: the psi_r parameter block at its bandwidth
// (validated SPD on the host).
template <int D>
__global__ void k_psi_setup(PsiBatchArgs a, double* __restrict__ prm) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= a.n_ds) return;
    const DsDev* dsp = a.rec[0];
    double gv[10];
    for (int t = 0; t < 10; ++t) gv[t] = a.Gv[0][t];
#pragma unroll
    for (int jj = 1; jj < KDEFFT_MAX_PSI_DS; ++jj)
        if (jj == j) {
            dsp = a.rec[jj];
#pragma unroll
            for (int t = 0; t < 10; ++t) gv[t] = a.Gv[jj][t];
        }
    psi_params<D>(gv, *dsp, a.prodP, prm + (int64_t)j * PRM);
}

hipError_t launch_psi_setup(const PsiBatchArgs& a, double* prm, hipStream_t s) {
    switch (a.d) {
        case 1: hipLaunchKernelGGL(k_psi_setup<1>, dim3(1), dim3(64), 0, s, a, prm); break;
        case 2: hipLaunchKernelGGL(k_psi_setup<2>, dim3(1), dim3(64), 0, s, a, prm); break;
        case 3: hipLaunchKernelGGL(k_psi_setup<3>, dim3(1), dim3(64), 0, s, a, prm); break;
        case 4: hipLaunchKernelGGL(k_psi_setup<4>, dim3(1), dim3(64), 0, s, a, prm); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Criterion assembly, one wavefront per candidate (see crit_finish); the
// npseudo constant-term candidates after the real ones store their term in
// their dataset's scalar block.  Work items of candidate c: c * nchunks + [0, nchunks).
// STEP: the value and the gradient go straight to the minimiser's update of the
// candidate (d = 2, 4 candidates, us per evaluation: assembly and update as two
// launches 14.5, together 4.3, with every load issued before the sums 3.9).
template <int D, bool STEP>
__global__ __launch_bounds__(64) void k_scv_final(int kind, const double* __restrict__ partial, int64_t nchunks, int ng,
                                                  const double* __restrict__ prm, int64_t ncand, int npseudo,
                                                  const double* __restrict__ grad_out, double* __restrict__ obj,
                                                  double* __restrict__ grad, MinStep step) {
    constexpr int Q = D * (D + 1) / 2;
    const int64_t h = blockIdx.x;
    if (h >= ncand + npseudo) return;
    const double* p = prm + h * PRM;
    if (h >= ncand) {
        double v[2];
        item_sums<1>(partial, h, -1, nchunks, ng, v);
        if (threadIdx.x == 0) static_cast<double*>(slot_ptr(p[S_FIN_SCAL]))[0] = v[0] * p[S_SCALE];
        return;
    }
    // with one dataset the constant term's place is known without reading the
    // candidate's record
    const int64_t c = npseudo == 0 ? -1 : npseudo == 1 ? ncand : (int64_t)p[S_PSEUDO];
    const ParamLanes pl(p);
    const double cscale = c >= 0 ? prm[c * PRM + S_SCALE] : 0.0;
    const bool grads = kind == FUN_SCV_OBJGRAD || kind == FUN_SCV_GRAD;
    double T[2 + Q], gv[Q];
    if constexpr (STEP) {
        const MinState<Q> now(step, h);
        item_sums<1 + Q>(partial, h, c, nchunks, ng, T);
        const double f = crit_finish<D>(kind, T, pl, T[1 + Q] * cscale, 1.0, true, gv);
        if (threadIdx.x == 0) min_step<Q>(step, h, now, f, gv);
        return;
    }
    item_sums<1 + Q>(partial, h, c, nchunks, ng, T);
    const double f = crit_finish<D>(kind, T, pl, T[1 + Q] * cscale, kind == FUN_SCV_GRAD ? grad_out[h] : 1.0,
                                    grads && grad != nullptr, gv);
    if (threadIdx.x != 0) return;
    if (kind != FUN_SCV_GRAD) obj[h] = f;
    if (grads && grad != nullptr)
#pragma unroll
        for (int i = 0; i < Q; ++i) grad[h * Q + i] = gv[i];
}

hipError_t launch_scv_final(int kind, int d, const double* partial, int64_t nchunks, const double* prm,
                            int64_t ncand, int npseudo, const double* grad_out, double* obj, double* grad,
                            const MinStep* step, hipStream_t s) {
    const int ng = ng_of(kind, d, 2);
    const dim3 grid((unsigned)(ncand + npseudo));
    if (step && kind != FUN_SCV_OBJGRAD) return hipErrorInvalidValue;
#define FINAL(DD)                                                                                                   \
    if (step)                                                                                                       \
        hipLaunchKernelGGL((k_scv_final<DD, true>), grid, dim3(64), 0, s, kind, partial, nchunks, ng, prm, ncand,   \
                           npseudo, grad_out, obj, grad, *step);                                                    \
    else                                                                                                            \
        hipLaunchKernelGGL((k_scv_final<DD, false>), grid, dim3(64), 0, s, kind, partial, nchunks, ng, prm, ncand,  \
                           npseudo, grad_out, obj, grad, MinStep{})
    switch (d) {
        case 1: FINAL(1); break;
        case 2: FINAL(2); break;
        case 3: FINAL(3); break;
        case 4: FINAL(4); break;
        default: return hipErrorInvalidValue;
    }
#undef FINAL
    return hipGetLastError();
}

// Position of each Kronecker-ordered 4-index (i, j, k, l) (first slowest)
// among the unique entries: sorted tuples in lexicographic order (Sec. 5).
template <int D>
struct Kron4 {
    int u[D * D * D * D];
    static constexpr Kron4 make() {
        Kron4 t{};
        int code[256] = {};
        int cnt = 0;
        for (int a = 0; a < D; ++a)
            for (int b = a; b < D; ++b)
                for (int c = b; c < D; ++c)
                    for (int e = c; e < D; ++e) code[((a * D + b) * D + c) * D + e] = cnt++;
        for (int f = 0; f < D * D * D * D; ++f) {
            int v[4] = {f / (D * D * D), (f / (D * D)) % D, (f / D) % D, f % D};
            for (int x = 0; x < 4; ++x)
                for (int y = 0; y + 1 < 4 - x; ++y)
                    if (v[y] > v[y + 1]) { const int tmp = v[y]; v[y] = v[y + 1]; v[y + 1] = tmp; }
            t.u[f] = code[((v[0] * D + v[1]) * D + v[2]) * D + v[3]];
        }
        return t;
    }
};

// Plug-in criterion, one thread per candidate:
//   PI(H) = n^-1 (4 pi)^{-d/2} |H|^{-1/2} + 1/4 sum_{ijkl} H_ij H_kl psi_ijkl,
//   grad_H = -1/2 (first term) H^{-1} + 1/2 sum_kl psi_ijkl H_kl,
// chained to vech(L) by dPI/dL = lower(2 grad_H L).
template <int D>
__global__ void k_pi(PiArgs a, const double* __restrict__ psi4, const double* __restrict__ vechL, int64_t ncand,
                     double* __restrict__ obj, double* __restrict__ grad, int32_t* __restrict__ status) {
    const int64_t h = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (h >= ncand) return;
    constexpr int d = D, q = D * (D + 1) / 2, NU = (D + 3) * (D + 2) * (D + 1) * D / 24;
    constexpr Kron4<D> K = Kron4<D>::make();
    int ds = 0;
    double n = a.n[0];
#pragma unroll
    for (int jj = 1; jj < KDEFFT_MAX_BATCH_DS; ++jj)
        if (jj < a.n_ds && h >= a.off[jj]) { ds = jj; n = a.n[jj]; }
    const double* ps = psi4 + (int64_t)ds * NU;
    double L[16], H[16];
    for (int i = 0; i < 16; ++i) L[i] = 0.0;
    int t = 0;
    bool sing = false;
    for (int jj = 0; jj < d; ++jj)
        for (int i = jj; i < d; ++i) {
            const double v = vechL[h * q + t++];
            L[i * 4 + jj] = v;
            if (!isfinite(v) || (i == jj && v == 0.0)) sing = true;
        }
    for (int i = 0; i < d; ++i)
        for (int k2 = 0; k2 < d; ++k2) {
            double s = 0.0;
            for (int k = 0; k < d; ++k) s += L[i * 4 + k] * L[k2 * 4 + k];
            H[i * 4 + k2] = s;
        }
    double ldet = 1.0;
    for (int k = 0; k < d; ++k) ldet *= fabs(L[k * 4 + k]);
    double c4 = 1.0;  // (4 pi)^{-d/2}
    for (int k = 0; k < d; ++k) c4 *= 0.28209479177387814347;
    const double first = sing ? 0.0 : c4 / (n * ldet);
    // M_ij = sum_kl psi_ijkl H_kl
    double Mq[16];
    double quad = 0.0;
#pragma unroll
    for (int i = 0; i < d; ++i)
#pragma unroll
        for (int j = 0; j < d; ++j) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < d; ++k)
#pragma unroll
                for (int l = 0; l < d; ++l) s += ps[K.u[((i * D + j) * D + k) * D + l]] * H[k * 4 + l];
            Mq[i * 4 + j] = s;
            quad += H[i * 4 + j] * s;
        }
    const double nan = __longlong_as_double(0x7ff8000000000000LL);
    if (status) status[h] = sing ? 1 : 0;
    if (obj) obj[h] = sing ? nan : first + 0.25 * quad;
    if (!grad) return;
    double Hinv[16];
    if (!sing) {
        chol_inv4<D>(L, Hinv);
    } else {
        for (int i = 0; i < 16; ++i) Hinv[i] = 0.0;
    }
    double gH[16];
    for (int i = 0; i < d; ++i)
        for (int j = 0; j < d; ++j) gH[i * 4 + j] = -0.5 * first * Hinv[i * 4 + j] + 0.5 * Mq[i * 4 + j];
    int o = 0;
    for (int j = 0; j < d; ++j)
        for (int i = j; i < d; ++i) {
            double s = 0.0;
            for (int k = 0; k < d; ++k) s += gH[i * 4 + k] * L[k * 4 + j];
            grad[h * q + o++] = sing ? nan : 2.0 * s;
        }
}

hipError_t launch_pi(const PiArgs& a, const double* psi4, const double* vechL, int64_t ncand, double* obj,
                     double* grad, int32_t* status, hipStream_t s) {
    const int64_t blocks = (ncand + 63) / 64;
    switch (a.d) {
        case 1: hipLaunchKernelGGL(k_pi<1>, dim3((unsigned)blocks), dim3(64), 0, s, a, psi4, vechL, ncand, obj, grad, status); break;
        case 2: hipLaunchKernelGGL(k_pi<2>, dim3((unsigned)blocks), dim3(64), 0, s, a, psi4, vechL, ncand, obj, grad, status); break;
        case 3: hipLaunchKernelGGL(k_pi<3>, dim3((unsigned)blocks), dim3(64), 0, s, a, psi4, vechL, ncand, obj, grad, status); break;
        case 4: hipLaunchKernelGGL(k_pi<4>, dim3((unsigned)blocks), dim3(64), 0, s, a, psi4, vechL, ncand, obj, grad, status); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// psi[h, g] = scale_h * sum over chunks (fixed order), one wavefront per
// (candidate, grid).
__global__ __launch_bounds__(64) void k_psi_final(const double* __restrict__ partial, int64_t nchunks, int ng,
                                                  const double* __restrict__ prm, int64_t ncand,
                                                  double* __restrict__ psi) {
    const int64_t e = blockIdx.x;
    if (e >= ncand * ng) return;
    const int64_t h = e / ng;
    const double v = chunk_sum(partial, h, nchunks, ng, (int)(e - h * ng)) * prm[h * PRM + S_SCALE];
    if (threadIdx.x == 0) psi[e] = v;
}

hipError_t launch_psi_final(const double* partial, const RowGeom& geo, int ng, const double* prm, int64_t ncand,
                            double* psi, hipStream_t s) {
    hipLaunchKernelGGL(k_psi_final, dim3((unsigned)(ncand * ng)), dim3(64), 0, s, partial, geo.nchunks, ng, prm,
                       ncand, psi);
    return hipGetLastError();
}

}  // namespace kdefft
