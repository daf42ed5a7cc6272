// Step 1 of Sec. 4: data bounds and linear binning into int64 fixed-point counts.
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "internal.h"
#include "params.h"

namespace kdefft {

// ------------------------------------------------------------------ bounds
// Per-block min/max of each column of X [n, D] into partial[block * 8 + k]
// (min) and partial[block * 8 + 4 + k] (max); min/max are exact, so the
// result does not depend on the reduction order.  partial may be pinned host
// memory (the host plans the grid: it reduces the partials itself, which saves
// a reducing launch and a copy before the wait).  Also clears zero16 16-byte
// words at zero_ptr (the binning's scratch), so the preparation needs no
// separate clearing launch.
template <int D>
__global__ __launch_bounds__(256) void k_bounds(const double* __restrict__ X, int64_t n,
                                                double* __restrict__ partial, uint4* __restrict__ zero_ptr,
                                                int64_t zero16, int32_t* __restrict__ n_out,
                                                double* __restrict__ scal) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < zero16; i += stride) zero_ptr[i] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x == 0 && threadIdx.x < 4) {   // the dataset's out-of-grid counter and scalar block
        if (n_out && threadIdx.x == 0) *n_out = 0;
        if (scal) scal[threadIdx.x] = 0.0;
    }
    double mn[D], mx[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
        mn[k] = INFINITY;
        mx[k] = -INFINITY;
    }
    // unrolled so that a thread's loads are in flight together
#pragma unroll 4
    for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < n; i += stride) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const double v = X[i * D + k];
            mn[k] = fmin(mn[k], v);
            mx[k] = fmax(mx[k], v);
        }
    }
    __shared__ double sw[4][8];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < D; ++k) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            mn[k] = fmin(mn[k], __shfl_xor(mn[k], off, 64));
            mx[k] = fmax(mx[k], __shfl_xor(mx[k], off, 64));
        }
        if (lane == 0) {
            sw[wid][k] = mn[k];
            sw[wid][4 + k] = mx[k];
        }
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)D) {
        const int k = threadIdx.x;
        double a = sw[0][k], b = sw[0][4 + k];
        for (int w = 1; w < 4; ++w) {
            a = fmin(a, sw[w][k]);
            b = fmax(b, sw[w][4 + k]);
        }
        partial[blockIdx.x * 8 + k] = a;
        partial[blockIdx.x * 8 + 4 + k] = b;
    }
}

hipError_t launch_bounds_partial(const double* X, int64_t n, int d, double* partial, int nblk, hipStream_t s,
                                 void* zero_ptr, size_t zero_bytes, int32_t* n_out, double* scal) {
    if (zero_bytes % 16 || (reinterpret_cast<uintptr_t>(zero_ptr) & 15)) return hipErrorInvalidValue;
    uint4* z = static_cast<uint4*>(zero_ptr);
    const int64_t z16 = (int64_t)(zero_bytes / 16);
    switch (d) {
        case 1: hipLaunchKernelGGL(k_bounds<1>, dim3(nblk), dim3(256), 0, s, X, n, partial, z, z16, n_out, scal); break;
        case 2: hipLaunchKernelGGL(k_bounds<2>, dim3(nblk), dim3(256), 0, s, X, n, partial, z, z16, n_out, scal); break;
        case 3: hipLaunchKernelGGL(k_bounds<3>, dim3(nblk), dim3(256), 0, s, X, n, partial, z, z16, n_out, scal); break;
        case 4: hipLaunchKernelGGL(k_bounds<4>, dim3(nblk), dim3(256), 0, s, X, n, partial, z, z16, n_out, scal); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ clearing
// Everything that a binning adds to, in one launch: words 64-bit words at p,
// the out-of-grid counter, and for a dataset on a given grid (hdr.rec set) its
// record, counter and scalar block.  A launch of its own for the counter or the
// record costs 2 us.
__global__ __launch_bounds__(256) void k_clear(uint64_t* __restrict__ p, int64_t words, int32_t* __restrict__ n_out,
                                               HeaderArgs hdr) {
    for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < words; i += gridDim.x * 256LL) p[i] = 0u;
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    if (n_out) *n_out = 0;
    if (hdr.rec) {
        *hdr.rec = hdr.val;
        for (int k = 0; k < 4; ++k) hdr.scal[k] = 0.0;
    }
}

hipError_t launch_clear(void* p, size_t bytes, int32_t* n_out, hipStream_t s, const HeaderArgs* hdr) {
    if (bytes % 8) return hipErrorInvalidValue;
    const int64_t words = (int64_t)(bytes / 8);
    int64_t blocks = (words + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    HeaderArgs h{};
    if (hdr) h = *hdr;
    hipLaunchKernelGGL(k_clear, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<uint64_t*>(p), words, n_out, h);
    return hipGetLastError();
}

// ------------------------------------------------------------------ linear binning
// Fixed-point contract (one thread per point):
//   t_k = (x_k - lo_k) / delta_k; skip unless 0 <= t_k <= M_k - 1
//   j_k = floor(t_k) (M_k - 1 -> M_k - 2); f_k = t_k - j_k; weights (1 - f_k, f_k)
//   corner weight = left-to-right product over axes; q = rint(w * 2^40)
//   the largest corner (lowest number on ties) takes 2^40 - sum of the others.
// Floating-point contraction is disabled so that every step is one IEEE
// operation, as on the host.
// slots != 0: the increments go to the corner slots of the last min(D, 3)
// axes (a record of 2^min(D, 3) int64 per cell), so that a point's 2^D
// increments fall in 2^max(D-3, 0) contiguous records; the count transform's
// first pass gathers the counts from the slots (exactly, in integers) while
// it reads them.  slots == 0: straight into the count grid.
//
// Scattered 64-bit atomics cost one memory-side request per distinct cache
// line per instruction, so after the per-point arithmetic the wavefront's
// 64 x 2^D corner increments are re-dealt through LDS: instruction `it` gives
// lane l the increment number it * 64 + l, i.e. point (it * 64 + l) / 2^D and
// corner (it * 64 + l) % 2^D in an order whose consecutive corners differ in
// the last (contiguous) axis, so neighbouring lanes add to adjacent bins of
// the grid (2^(D-1) cache lines per point), or, with the corner slots, to one
// record per 2^min(D, 3) lanes (one cache line per point, two for D = 4).
// Grid origin and spacing from the data bounds (per-block partials of the
// bounds kernel), by the same IEEE steps and order as the host planner:
// lo = min - pad, hi = max + pad, hi = lo + 1 for a degenerate axis,
// delta = (hi - lo) / (M - 1); non-finite data give a NaN spacing, so every
// point counts as out of the grid.  Called by all threads of a block.
template <int D>
__device__ __forceinline__ void grid_from_bounds(const HeaderArgs& h, double* lo, double* delta, int* reach) {
#pragma clang fp contract(off)
    __shared__ double scratch[32], red[8], sg[8];
    reduce_bounds(h.partial, h.nblk, D, scratch, red);
    if (threadIdx.x < (unsigned)D) {
        const int k = threadIdx.x;
        const double nan = __longlong_as_double(0x7ff8000000000000LL);
        const double l = red[k] - h.pad[k];
        double hi = red[4 + k] + h.pad[k];
        if (!isfinite(l) || !isfinite(hi)) {
            sg[k] = nan;
            sg[4 + k] = nan;
        } else {
            if (!(hi > l)) hi = l + 1.0;
            sg[k] = l;
            sg[4 + k] = (hi - l) / (double)(h.g.M[k] - 1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < D; ++k) {
        lo[k] = sg[k];
        delta[k] = sg[4 + k];
        // the counts' nodes span at most two spacings more than the data do (a
        // non-finite span keeps the whole axis)
        const double span = floor((red[4 + k] - red[k]) / delta[k]) + 2.0;
        reach[k] = span < (double)(h.g.M[k] - 1) ? (int)span : h.g.M[k] - 1;
    }
}

// Origin and spacing from the bound partials into g; block 0 writes the
// dataset record.  Called by all threads of a block.
template <int D>
__device__ __forceinline__ void dataset_header(const HeaderArgs& hdr, kdefft_grid& g) {
    int reach[D];
    grid_from_bounds<D>(hdr, g.lo, g.delta, reach);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        DsDev v = hdr.val;
        for (int k = 0; k < D; ++k) {
            v.lo[k] = g.lo[k];
            v.delta[k] = g.delta[k];
            v.reach[k] = reach[k];
        }
        *hdr.rec = v;
    }
}

// One point's increments (the contract above) and the flat index of its lowest
// corner; false when the point lies outside the grid (q and fb then unset).
// Corner b: bit k set = upper node along axis k.  The integers are formed as
// doubles, exactly: w * 2^40 is a scaling, below 2^52, so adding 2^52 rounds
// it to the nearest integer (ties to even); differences and sums of these
// integers stay below 2^53; and 2^52 + q holds q in its low mantissa bits.
template <int D, class I>
__device__ __forceinline__ bool point_increments(const double* x, const kdefft_grid& g, const I* stride, long long* q,
                                                 I& fb) {
#pragma clang fp contract(off)
    constexpr int NC = 1 << D;
    const double one_q = 1099511627776.0, big = 4503599627370496.0;   // 2^40, 2^52
    double w0[D], w1[D];
    I f0 = 0;
    bool ok = true;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const double t = (x[k] - g.lo[k]) / g.delta[k];
        ok = ok && (t >= 0.0) && (t <= (double)(g.M[k] - 1));
        // M - 1 -> M - 2 (and outside the grid a value that an int holds)
        const double jf = fmax(fmin(floor(t), (double)(g.M[k] - 2)), 0.0);
        const double f = t - jf;
        w0[k] = 1.0 - f;
        w1[k] = f;
        f0 += (I)(int)jf * stride[k];
    }
    fb = f0;
    double v[NC], top, sum;
#pragma unroll
    for (int b = 0; b < NC; ++b) {
        double w = (b & 1) ? w1[0] : w0[0];
#pragma unroll
        for (int k = 1; k < D; ++k) w = w * (((b >> k) & 1) ? w1[k] : w0[k]);
        v[b] = fma(w, one_q, big) - big;
        top = b ? fmax(top, v[b]) : v[b];
        sum = b ? sum + v[b] : v[b];
    }
    const double fix = one_q - (sum - top);
    bool taken = false;
#pragma unroll
    for (int b = 0; b < NC; ++b) {
        const bool m = v[b] == top && !taken;
        taken = taken || m;
        q[b] = __double_as_longlong((m ? fix : v[b]) + big) & 0xfffffffffffffLL;
    }
    return ok;
}

// hdr.partial set: the dataset header is computed here, not by a separate
// launch: every block derives the grid origin and spacing from the bound
// partials (grid_from_bounds), and block 0 writes the dataset record.
template <int D>
__global__ __launch_bounds__(256) void k_linbin(const double* __restrict__ X, int64_t n, kdefft_grid g,
                                                unsigned long long* __restrict__ counts,
                                                int32_t* __restrict__ n_out, int slots, HeaderArgs hdr) {
#pragma clang fp contract(off)
    constexpr int NC = 1 << D;
    __shared__ long long qs[256 * NC];   // increments, per wavefront in issue order
    __shared__ int64_t fbs[256];         // flat index of each point's lowest corner
    if (hdr.partial) dataset_header<D>(hdr, g);   // block-uniform
    int64_t stride[D];
    stride[D - 1] = 1;
#pragma unroll
    for (int k = D - 2; k >= 0; --k) stride[k] = stride[k + 1] * g.M[k + 1];
    const int lane = threadIdx.x & 63, w0ff = threadIdx.x & ~63;
    for (int64_t i0 = blockIdx.x * 256LL; i0 < n; i0 += (int64_t)gridDim.x * 256) {   // block-uniform
        const int64_t i = i0 + threadIdx.x;
        long long q[NC];
#pragma unroll
        for (int b = 0; b < NC; ++b) q[b] = 0;
        int64_t fb = 0;
        if (i < n) {
            double x[D];
#pragma unroll
            for (int k = 0; k < D; ++k) x[k] = X[i * D + k];
            if (!point_increments<D>(x, g, stride, q, fb)) {
#pragma unroll
                for (int b = 0; b < NC; ++b) q[b] = 0;
                if (n_out) atomicAdd(n_out, 1);
            }
        }
        // issue order c = bit-reversed b: bit 0 of c is the last axis
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            int c = 0;
#pragma unroll
            for (int k = 0; k < D; ++k) c |= ((b >> k) & 1) << (D - 1 - k);
            qs[w0ff * NC + lane * NC + c] = q[b];
        }
        fbs[threadIdx.x] = fb;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < NC; ++it) {
            const int a = it * 64 + lane;
            const int pnt = a / NC, c = a % NC;
            const long long v = qs[w0ff * NC + a];
            if (v != 0) {
                if (slots) {
                    // record: the lowest corner moved along the unslotted
                    // leading axes of corner c; slot: c's bits of the slotted axes
                    constexpr int NSA = slot_axes(D), NS = corner_slots(D);
                    int64_t off = 0;
#pragma unroll
                    for (int k = 0; k + NSA < D; ++k) off += ((c >> (D - 1 - k)) & 1) * stride[k];
                    atomicAdd(counts + (fbs[w0ff + pnt] + off) * NS + (c & (NS - 1)), (unsigned long long)v);
                } else {
                    int64_t off = 0;
#pragma unroll
                    for (int k = 0; k < D; ++k) off += ((c >> (D - 1 - k)) & 1) * stride[k];
                    atomicAdd(counts + fbs[w0ff + pnt] + off, (unsigned long long)v);
                }
            }
        }
        __syncthreads();
    }
}

// The same increments summed in LDS first.  The scattered atomics above run
// at the memory side's rate of about 11e9 records a second, whatever the
// grid's size; a sample much larger than its grid is cheaper to add up on the
// compute units.  A block holds one band of BAND consecutive nodes and adds
// its part of the points to it, skipping the corners of other bands, then adds
// the band to the counts, neighbouring lanes to neighbouring nodes.  Bound by
// the per-point arithmetic, about 135 instructions for d = 2, repeated once
// per band: 2e6 points on 256 x 256 nodes (4 bands), whole preparation 205 ->
// 74 us.  (Passing on only the points that reach the band, through a queue per
// wavefront, measured the same: the middle bands take half of the points.)
// The bands of one part of the points run on one XCD (blocks b and b + 8 share
// it), which reads the part from memory once.  Counts as above, bit for bit:
// the sums are integers.  The count grid must be zero on entry.
constexpr int BAND = 20416;   // 160 KB less the header's scratch
template <int D>
__global__ __launch_bounds__(1024) void k_linbin_bands(const double* __restrict__ X, int64_t n, kdefft_grid g,
                                                       unsigned long long* __restrict__ counts,
                                                       int32_t* __restrict__ n_out, int nodes, int band_nodes,
                                                       int nbands, int64_t part_points, HeaderArgs hdr) {
    constexpr int NC = 1 << D, U = D < 3 ? 4 : 2;
    __shared__ unsigned long long acc[BAND];
    if (hdr.partial) {
        dataset_header<D>(hdr, g);
        __syncthreads();
    }
    const int band = (int)(blockIdx.x / 8) % nbands;
    const int64_t part = (int64_t)(blockIdx.x / (8 * nbands)) * 8 + blockIdx.x % 8;
    const int first = band * band_nodes, len = min(band_nodes, nodes - first);
    for (int i = threadIdx.x; i < len; i += 1024) acc[i] = 0;
    int stride[D];
    stride[D - 1] = 1;
#pragma unroll
    for (int k = D - 2; k >= 0; --k) stride[k] = stride[k + 1] * g.M[k + 1];
    __syncthreads();
    const int64_t p0 = part * part_points, p1 = p0 + part_points < n ? p0 + part_points : n;
    int out = 0;
    for (int64_t i0 = p0 + threadIdx.x; i0 < p1; i0 += 1024 * U) {
        double x[U][D];   // U points' loads in flight
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + 1024 * u < p1 ? i0 + 1024 * u : i0;
#pragma unroll
            for (int k = 0; k < D; ++k) x[u][k] = X[i * D + k];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + 1024 * u >= p1) break;
            long long q[NC];
            int fb;
            const bool ok = point_increments<D>(x[u], g, stride, q, fb);
            out += !ok;
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                int off = -first;
#pragma unroll
                for (int k = 0; k < D; ++k) off += ((b >> k) & 1) * stride[k];
                const int c = fb + off;
                if (ok && (unsigned)c < (unsigned)len) atomicAdd(&acc[c], (unsigned long long)q[b]);
            }
        }
    }
    if (out && band == 0 && n_out) atomicAdd(n_out, out);
    __syncthreads();
    for (int i = threadIdx.x; i < len; i += 1024) {
        const unsigned long long v = acc[i];
        if (v) atomicAdd(counts + first + i, v);
    }
}

// Bands or scattered atomics.  A block's flush costs its band's nodes, the
// scattered records n; the repeated arithmetic costs n times the bands.  Whole
// preparations, us, scattered -> bands (normal data): d = 1, M = 500: n = 1e4
// 31.5 -> 31.3, 1e5 76 -> 34, 2e6 1103 -> 44; d = 2, M = 200 (2 bands): 5e4
// 37.5 -> 39.0, 1e5 41.9 -> 42.1, 2e5 52.8 -> 46.4, 2e6 218 -> 68; M = 300
// (5 bands): 2e5 70 -> 76, 5e5 85 -> 80; d = 3, M = 27 (1 band): 2e4 47.9 ->
// 47.8, 1e5 57 -> 49; M = 54 (8 bands): 1e5 87.4 -> 87.8, 2e6 215 -> 179;
// d = 4, M = 16 (4 bands): 1e4 75 -> 68, 2e6 739 -> 159.  Hence bands from
// 10000 points and from 3 points a node for d <= 2, one for d = 3 and a
// quarter for d = 4 (2^d increments a point).
constexpr int MAX_BANDS = 8;
bool linbin_in_bands(int64_t n, const kdefft_grid& g) {
    int64_t nodes = 1;
    for (int k = 0; k < g.d; ++k) nodes *= g.M[k];
    return nodes <= MAX_BANDS * BAND && n >= 10000 && (g.d == 4 ? 4 * n : n) >= (g.d <= 2 ? 3 * nodes : nodes);
}

hipError_t launch_linbin_bands(const double* X, int64_t n, const kdefft_grid& g, int64_t* counts, int32_t* n_out,
                               hipStream_t s, const HeaderArgs* hdr) {
    int64_t nodes = 1;
    for (int k = 0; k < g.d; ++k) nodes *= g.M[k];
    if (nodes > MAX_BANDS * BAND) return hipErrorInvalidValue;
    const int nbands = (int)((nodes + BAND - 1) / BAND), band_nodes = (int)((nodes + nbands - 1) / nbands);
    // parts in eights (one per XCD), at most one block per compute unit and at
    // least 1024 points each (8192: d = 4, M = 8, n = 1e5 58 us, 1024: 44 us)
    int64_t parts = 256 / nbands / 8 * 8;
    while (parts > 8 && n / parts < 1024) parts -= 8;
    const int64_t part_points = (n + parts - 1) / parts;
    HeaderArgs h{};
    if (hdr) h = *hdr;
    const dim3 grid((unsigned)(parts * nbands));
    auto* c = reinterpret_cast<unsigned long long*>(counts);
    switch (g.d) {
        case 1: hipLaunchKernelGGL(k_linbin_bands<1>, grid, dim3(1024), 0, s, X, n, g, c, n_out, (int)nodes, band_nodes, nbands, part_points, h); break;
        case 2: hipLaunchKernelGGL(k_linbin_bands<2>, grid, dim3(1024), 0, s, X, n, g, c, n_out, (int)nodes, band_nodes, nbands, part_points, h); break;
        case 3: hipLaunchKernelGGL(k_linbin_bands<3>, grid, dim3(1024), 0, s, X, n, g, c, n_out, (int)nodes, band_nodes, nbands, part_points, h); break;
        case 4: hipLaunchKernelGGL(k_linbin_bands<4>, grid, dim3(1024), 0, s, X, n, g, c, n_out, (int)nodes, band_nodes, nbands, part_points, h); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_linbin_slots(const double* X, int64_t n, const kdefft_grid& g, int64_t* slots, int32_t* n_out,
                               hipStream_t s, const HeaderArgs* hdr) {
    int64_t blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    auto* c = reinterpret_cast<unsigned long long*>(slots);
    HeaderArgs h{};
    if (hdr) h = *hdr;
    switch (g.d) {
        case 1: hipLaunchKernelGGL(k_linbin<1>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 1, h); break;
        case 2: hipLaunchKernelGGL(k_linbin<2>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 1, h); break;
        case 3: hipLaunchKernelGGL(k_linbin<3>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 1, h); break;
        case 4: hipLaunchKernelGGL(k_linbin<4>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 1, h); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_linbin(const double* X, int64_t n, const kdefft_grid& g, int64_t* counts, int32_t* n_out,
                         hipStream_t s) {
    int64_t blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    if (blocks < 1) blocks = 1;
    auto* c = reinterpret_cast<unsigned long long*>(counts);
    const HeaderArgs h{};
    switch (g.d) {
        case 1: hipLaunchKernelGGL(k_linbin<1>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 0, h); break;
        case 2: hipLaunchKernelGGL(k_linbin<2>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 0, h); break;
        case 3: hipLaunchKernelGGL(k_linbin<3>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 0, h); break;
        case 4: hipLaunchKernelGGL(k_linbin<4>, dim3((unsigned)blocks), dim3(256), 0, s, X, n, g, c, n_out, 0, h); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace kdefft
