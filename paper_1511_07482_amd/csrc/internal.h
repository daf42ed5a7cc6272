// Internal interface between the C-ABI layer (api.cpp) and the HIP kernels.
// Nothing here is exported.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/kdefft.h"

namespace kdefft {

constexpr int PRM = 68;     // doubles per candidate parameter block
constexpr int NT_DEF = 256;  // threads per block of the simple kernels

// Parameter block layout (float64 slots) shared by setup, row and finalize kernels.
// Matrices use row stride 4.
//   psi:  [0,16) P = G^{-1}   [16] c = (-1)^r (2pi)^{-d/2}|G|^{-1/2}
//   scv:  [0,16) P1 = (2H+2G)^{-1}  [16,32) P2 = (H+2G)^{-1}  [32] c1  [33] c2
//   both: [38] alag pointer bits  [39] wmix pointer bits  [40,44) delta  [44] n  [45] 1/(n^2 prod P)
//         [46] constant term  [47] singular flag  [48,64) L (scv) / P3 (plain scv)
//   criteria: [34] first (closed-form) term  [35] r of eta_r  [36] sign (-1)^r
//         [37] SCV: the candidate index whose objective sum is the dataset's constant phi_{2G} term
enum Slot { S_P1 = 0, S_C = 16, S_P2 = 16, S_C1 = 32, S_C2 = 33, S_FIRST = 34, S_R = 35, S_SIGN = 36, S_PSEUDO = 37,
            S_ALAG = 38,
            S_WMIX = 39, S_DELTA = 40, S_N = 44, S_SCALE = 45, S_CONST = 46, S_SING = 47, S_L = 48,
            S_FIN_SCAL = 64 };   // constant-term candidates: the dataset's scalar block


// Per-dataset record kept in the dataset's own device buffer (written by a
// kernel at prepare time); batched calls pass pointers to these records.
struct DsDev {
    const double2* wmix;
    const double* alag;
    const double* scal;
    double n;
    double lo[4];      // grid origin and spacing (lo, delta contiguous: the
    double delta[4];   // binning kernel reads them from here on the device path)
    double G[16];   // pilot, row stride 4
    int32_t reach[4];   // largest |lag| per axis at which the autocorrelation can differ from zero
};

// Kernel-argument views of a batch (no host-to-device copies per call).
struct ScvBatchArgs {
    int n_ds;
    int d;
    int crit;   // KDEFFT_CRIT_*
    int r;      // order of eta_r (0 for SCV)
    double prodP;
    const DsDev* rec[KDEFFT_MAX_BATCH_DS];
    int64_t off[KDEFFT_MAX_BATCH_DS + 1];
};
struct PsiBatchArgs {
    int n_ds;
    int d;
    int r;
    double prodP;
    const DsDev* rec[KDEFFT_MAX_PSI_DS];
    double Gv[KDEFFT_MAX_PSI_DS][10];   // vech (columns of the lower triangle)
};
struct PiArgs {
    int n_ds;
    int d;
    double n[KDEFFT_MAX_BATCH_DS];
    int64_t off[KDEFFT_MAX_BATCH_DS + 1];
};
// One parameter block passed by value.
struct ParamBlock {
    double v[64];
};

// What the column walk (cols.h) needs to compute a candidate's parameters in
// its own launch: each work item's block factors its candidate's matrices from
// vechL and the dataset records into LDS, and the block of the candidate's
// first item also stores the slots the final kernel reads to prm_out (and the
// status).
struct ScvSetup {
    int npseudo;
    int64_t ncand;
    const double* vechL;
    int32_t* status;
    double* prm_out;
    ScvBatchArgs a;
};

// Geometry of the row decomposition of the lag grid used by the batched kernels.
struct RowGeom {
    int d;
    int M[4];
    int P[4];
    int64_t nrows;     // rows of the half lag set with nonzero kernel values
    int64_t chunk;     // rows per work item
    int64_t nchunks;   // work items per candidate
    int Q;             // P[d-1]/2 + 1
};

// Kinds of kernel families generated on the lag grid.
// FUN_SCV_* serve every criterion with two Gaussians and a Hessian gradient
// (SCV, LSCV); FUN_ETA1 / FUN_ETA2 are the scalar eta_r families (Q_r, LSCV_r).
enum FunKind { FUN_PSI = 0, FUN_SCV_OBJ = 1, FUN_SCV_OBJGRAD = 2, FUN_SCV_GRAD = 3, FUN_ETA1 = 4, FUN_ETA2 = 5 };

int ng_of(int kind, int d, int r);   // number of kernel grids of a family

// -------------------------------------------------------------- launchers
// All return hipSuccess or the first HIP error; they only enqueue work.
hipError_t twiddles(const double2** out);  // per-device table e^{-2 pi i m/4096} + N-point subsets

// Data bounds: per-block partials (nblk blocks; 8 doubles each, min[4], max[4]),
// clearing zero_bytes (a multiple of 16, 16-byte aligned) at zero_ptr on the way.
hipError_t launch_bounds_partial(const double* X, int64_t n, int d, double* partial, int nblk, hipStream_t s,
                                 void* zero_ptr, size_t zero_bytes, int32_t* n_out = nullptr, double* scal = nullptr);
// Binning into the count grid (zero on entry).
hipError_t launch_linbin(const double* X, int64_t n, const kdefft_grid& g, int64_t* counts,
                         int32_t* n_out, hipStream_t s);
// Binning into corner slots over the last min(d, 3) axes: a record of
// S = 2^min(d, 3) int64 per cell of the count grid (slots: S * prod M int64,
// zero on entry).  A point adds its 2^d corner weights to
// 2^(d-3) records for d = 4 (one per node of axis 0: the cell of the lowest
// corner moved along axis 0 for the upper one), to one record otherwise,
// slot s of a record taking the corner's nodes along the slotted axes (bit j
// of s: upper along axis d-1-j).  A point's increments thus fall in
// 2^max(d-3, 0) contiguous records (one cache line each) instead of 2^(d-1)
// pairs of grid cells.  The count transform's first pass (fft_prepare_nd with
// slots) gathers each count exactly from S nearby slots:
// count(i) = sum over s of slot s of record i - e(s).
__host__ __device__ constexpr int slot_axes(int d) { return d < 3 ? d : 3; }
__host__ __device__ constexpr int corner_slots(int d) { return 1 << slot_axes(d); }
struct HeaderArgs;
// hdr (may be NULL): with hdr->partial set, the binning launch also computes
// the grid from the bound partials and writes the dataset header (block 0).
hipError_t launch_linbin_slots(const double* X, int64_t n, const kdefft_grid& g, int64_t* slots, int32_t* n_out,
                               hipStream_t s, const HeaderArgs* hdr = nullptr);
// Binning straight into the count grid (zero on entry) by bands of nodes in
// LDS: for the samples and grids that linbin_in_bands accepts.
bool linbin_in_bands(int64_t n, const kdefft_grid& g);
hipError_t launch_linbin_bands(const double* X, int64_t n, const kdefft_grid& g, int64_t* counts, int32_t* n_out,
                               hipStream_t s, const HeaderArgs* hdr = nullptr);

// A dataset's record and what to write with it.  partial set: the grid origin
// and spacing come from the data bounds, in the binning launch -- lo = min - pad,
// hi = max + pad, hi = lo + 1 for a degenerate axis, delta = (hi - lo)/(M - 1),
// the same IEEE steps as the host planner.
struct HeaderArgs {
    DsDev* rec;
    DsDev val;
    const double* partial;   // per-block bound partials of the data (or NULL: keep val's grid)
    int nblk;
    kdefft_grid g;
    double pad[4];
    double* scal;
};
// Clears what a binning adds to: bytes (a multiple of 8) at p, the counter
// n_out (may be NULL); hdr (may be NULL): a dataset's record is written and its
// scalar block cleared too.
hipError_t launch_clear(void* p, size_t bytes, int32_t* n_out, hipStream_t s, const HeaderArgs* hdr = nullptr);

// Transforms along all axes but the first of arrays of slices (fft.hip).
hipError_t fft_slices_forward(const double* in, double2* out, const kdefft_grid& g, int64_t slices, hipStream_t s);
hipError_t fft_slices_inverse(double2* buf, const kdefft_grid& g, int64_t slices, hipStream_t s);
// spec = R2C of the counts: src, or gathered from the binning's corner slots
// in src (slots set; then also written to counts).
hipError_t fft_counts_nd(const int64_t* src, int slots, int64_t* counts, double2* spec, const kdefft_grid& g,
                         hipStream_t s);
// FFT-stage schedules of the count transform (launch shapes and radix order
// of its passes; fft.hip FS_*): fs in [0, FFT_SCHEDULES), 0 the default.
constexpr int FFT_SCHEDULES = 6;
// Count spectrum of a prepared dataset: spec = R2C(czp); wmix = |spec|^2
// transformed forward along the leading axes.  The first pass reads the int64
// counts directly: src is the count grid itself (slots = 0) or the corner
// slots of the binning (slots = 1), from which it gathers the counts exactly
// and also writes them to counts.
// reach (may be NULL): set to M - 1 per axis (counts that need not be those the
// dataset was binned with).
hipError_t fft_prepare_nd(const int64_t* src, int slots, int64_t* counts, double2* spec, double2* wmix,
                          const kdefft_grid& g, hipStream_t s, int fs, int32_t* reach = nullptr);
// alag = inverse transform of |C|^2 = prod P times the count autocorrelation,
// computed from the mixed spectrum (rows at negated leading indices).
hipError_t fft_autocorr_nd(const double2* wmix, double* alag, const kdefft_grid& g, hipStream_t s, int fs);

// Paper-literal path.  Step 2: the kernel grids of entries [first, first + nent)
// of a family at the slices l_0 = 0..m-1 (m = M_0; d = 1: the whole row) of the
// circular layout, kreal [nent, m, P_1, .., P_{d-1}]; the support is |l_k| < g.M[k].
hipError_t launch_kgrid_psi(double* kreal, const kdefft_grid& g, int m, int r, const ParamBlock& prm, int first,
                            int nent, hipStream_t s);
hipError_t launch_kgrid_scv(double* kreal, const kdefft_grid& g, int m, const ParamBlock& prm, int first, int nent,
                            hipStream_t s);
// Steps 3 and 4 (conv.hip): transform of kreal into K [nent, m, P_1, .., Q],
// product with the count spectrum C, inverse, and out[e] = scale * sum over the
// nodes of counts times convolution.  mk: the kernels' support along axis 0
// (l_0 < mk).  partial: nent * conv_blocks(g) values.
int conv_blocks(const kdefft_grid& g);
hipError_t conv_sums(const kdefft_grid& g, int mk, int nent, double* kreal, double2* K, const double2* C,
                     const int64_t* counts, double* partial, double scale, double* out, hipStream_t s);
hipError_t launch_scv_plain_final(const double* sums, const ParamBlock& fin, int d, double* out,
                                  hipStream_t s);

// Batched row kernels.
struct RowLaunch {
    int variant;        // compiled launch variant (rows per iteration, radix schedule)
    int grid_blocks;    // persistent grid size; 0 = occupancy x CUs, -1 = one block per item
};
hipError_t launch_rows(int kind, int d, int r, const RowGeom& geo, const double* prm, int64_t ncand,
                       double* partial, const RowLaunch& rl, hipStream_t s);
int rows_per_iter(int kind, int d, int r, int N, int variant);
// compiled lag-kernel layout for last-axis length N (0 = unsupported N)
int lag_layout(int N, int moments, int* run_len, int* runs_per_seg, int* rows_per_pass);
// 0-2: spectral (per-candidate FFT); 3, 4: lag domain (4: scaled walk of rising
// runs); 5, 6: as 3, 4 with only the live runs of each row dealt to the threads
constexpr int ROW_VARIANTS = 7;
// ncand real candidates, then npseudo constant-term candidates (SCV: one per
// dataset); wc (may be NULL) receives the candidates' live run counts.
hipError_t launch_scv_setup(const double* vechL, const ScvBatchArgs& a, int64_t ncand, int npseudo, double* prm,
                            int32_t* status, const RowGeom& geo, int32_t* wc, hipStream_t s);
hipError_t launch_psi_setup(const PsiBatchArgs& a, double* prm, hipStream_t s);
// State of a batch of minimisations (minstep.h): per candidate
// min_state_doubles(q) doubles and min_state_ints() int32, the criterion's
// status (may be NULL) and the trial points.
struct MinStep {
    double tol;
    double* st;
    int32_t* ist;
    const int32_t* stt;
    double* xt;
};
// step (may be NULL; FUN_SCV_OBJGRAD): the values and gradients go to one
// update of the minimiser instead of obj and grad.
hipError_t launch_scv_final(int kind, int d, const double* partial, int64_t nchunks,
                            const double* prm, int64_t ncand, int npseudo, const double* grad_out,
                            double* obj, double* grad, const MinStep* step, hipStream_t s);
hipError_t launch_psi_final(const double* partial, const RowGeom& geo, int ng,
                            const double* prm, int64_t ncand, double* psi, hipStream_t s);

// batched quasi-Newton minimiser (minimize.hip)
int min_state_doubles(int q);
int min_state_ints();
hipError_t launch_min_init(int64_t B, int q, const double* x0, double* xt, int32_t* ist, hipStream_t s);
hipError_t launch_min_step(int64_t B, int q, const MinStep& a, const double* ft, const double* gt, hipStream_t s);
hipError_t launch_min_final(int64_t B, int q, const double* st, const int32_t* ist, double* x_out, double* f_out,
                            int32_t* info, hipStream_t s);
hipError_t launch_pi(const PiArgs& a, const double* psi4, const double* vechL, int64_t ncand, double* obj,
                     double* grad, int32_t* status, hipStream_t s);

// Column walk (cols.h): the SCV / LSCV families (variants 5, 6), psi_r
// (variants from 3 on) and the eta_r families of low order (cols_eta_ok).
struct ColGeom {
    int M[4];
    int P[4];
    int n0;            // d >= 3: groups of axis-0 lags (nchunks is a multiple)
    int64_t nchunks;   // work items per candidate
};
// ng: outputs per item; scv: the batch may have to fit the fixed scratch of the
// call without a workspace.
// max_chunks: work items per candidate that the partial sums have room for.
ColGeom cols_geom(const kdefft_grid& g, int64_t ncand, int ng, bool scv, int64_t max_chunks = INT64_MAX);
bool cols_eta_ok(int d, int r);
// floor(u / d) for u >= 0 and rd = 1 / d: exact while the roundings of (u + 1/2) rd
// stay below 1 / (2 d), in float for u < 2^22, in double for all int.  d <= 3: the
// units of a candidate stay below 2^21 (prod P <= 2^30, P <= 4096).  d = 4: a part has up
// to 2^23, where the last two axes are short, the others long and the
// candidates so many that the axis-0 groups are few.
template <int D>
using ColRecip = std::conditional_t<D == 4, double, float>;
template <class R>
__host__ __device__ inline int col_quot(int u, R rd) { return (int)(((R)u + (R)0.5) * rd); }
hipError_t launch_cols_scv(int kind, int d, const ColGeom& geo, const ScvSetup& setup, int64_t nitems,
                           double* partial, int grid_blocks, hipStream_t s);
hipError_t launch_cols_eta(int kind, int d, int r, const ColGeom& geo, const ScvSetup& setup, int64_t nitems,
                           double* partial, int grid_blocks, hipStream_t s);
// One block per item, then one per dataset; prm: PRM doubles per dataset.
hipError_t launch_cols_psi(const ColGeom& geo, const PsiBatchArgs& a, int grid_blocks, double* prm, double* partial,
                           double* psi, hipStream_t s);

RowGeom make_geom(const kdefft_grid& g, int kind, int r, int64_t ncand, int variant, int64_t max_chunks = INT64_MAX);

// The work items of a criterion launch over nc candidates (real and
// constant-term ones): the column walk's or the row kernels' geometry.
struct CritWalk {
    bool cols;
    ColGeom col;
    RowGeom row;
    int64_t nchunks;
};
// room: doubles of partial sums.  kind, r: kernel family and criterion order.
CritWalk crit_walk(const kdefft_grid& g, int kind, int r, int variant, int64_t nc, int64_t room);
// Doubles of partial sums in the workspace of a batch of B candidates.
int64_t crit_room(const kdefft_grid& g, int64_t B);

// Host helpers of the C-ABI layer shared with other units: record an error
// (returned code, message for kdefft_last_error_detail), and the workspace
// bytes kdefft_scv_batch needs for a batch (validates the datasets and offsets).
int set_error(int code, const char* msg);
int scv_batch_ws_need(const kdefft_dataset* ds, int n_ds, const int64_t* off, size_t* need);

}  // namespace kdefft
