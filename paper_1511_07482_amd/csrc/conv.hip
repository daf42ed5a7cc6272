// The paper's steps 3 and 4 (Sec. 4, Eq. (22)-(24)) for several kernel grids at
// once: the convolution with the counts along axis 0 (transform, product with
// the count spectrum, inverse transform in one pass) and the inverse transform
// of the last axis with the count-weighted sum taken from its rows.
//
// Only half of a kernel grid is formed: k(-l) = k(l), so once the other axes are
// transformed the slice at lag -l_0 is the conjugate of the slice at l_0.  The
// buffers hold the slices l_0 = 0..M_0-1 of each grid, and after the axis-0 pass
// the convolution at the nodes i_0 = 0..M_0-1 in the same places; the later
// passes visit the nodes inside the counts' box only.
//
// Bound: the latency of a few small passes (d = 2, M = 256: 1 MB read and written
// per grid and pass).  psi_4 at n = 1e5, M = 256 (five grids), kernel grids to sums:
// 35 launches and 190 us one grid and one step at a time, 5 launches and 44 us
// like this (whole call 274 -> 102 us).
#include <hip/hip_runtime.h>

#include "dev_common.h"
#include "internal.h"

namespace kdefft {

// Columns per tile of an axis-0 pass of length N: what fits about 64 KiB.
template <int N>
constexpr int conv_cols() { return 4096 / (N + 1) >= 8 ? 8 : 4096 / (N + 1) >= 4 ? 4 : 4096 / (N + 1) >= 2 ? 2 : 1; }

// Entry blockIdx.y, columns [T blockIdx.x, +T): K holds slices [0, m) of inner
// values, the first mk of them the kernel's lags l_0 >= 0.
template <int N, int NT, int T>
__global__ __launch_bounds__(NT) void k_conv_axis0(double2* __restrict__ K, const double2* __restrict__ C,
                                                   int64_t inner, int mk, int m, const double2* __restrict__ tw) {
    constexpr int PS = T > 1 ? N + 1 : N;
    __shared__ double2 lds[T * PS];
    __shared__ double2 twl[N];
    TwiddleCopy<N, NT> twc;
    twc.fetch(tw);
    const int64_t i0 = (int64_t)blockIdx.x * T;
    double2* base = K + (int64_t)blockIdx.y * m * inner + i0;
    const double2* cb = C + i0;
    constexpr int PE = (N * T + NT - 1) / NT;   // unrolled: the loads in flight together
#pragma unroll
    for (int u = 0; u < PE; ++u) {
        const int e = threadIdx.x + u * NT;
        if ((N * T) % NT == 0 || e < N * T) {
            const int t = e % T, p = e / T;
            const int l = p < mk ? p : (N - p < mk ? N - p : -1);   // |lag| of position p, or a zero slot
            double2 v = make_double2(0.0, 0.0);
            if (l >= 0 && i0 + t < inner) v = base[(int64_t)l * inner + t];
            lds[t * PS + p] = p < mk ? v : c_conj(v);
        }
    }
    twc.store(twl, tw);
    __syncthreads();
    fft_lds<N, T, NT, -1, 0, N>(lds, PS, twl);
#pragma unroll
    for (int u = 0; u < PE; ++u) {
        const int e = threadIdx.x + u * NT;
        if ((N * T) % NT == 0 || e < N * T) {
            const int t = e % T, p = e / T;
            if (i0 + t < inner) lds[t * PS + p] = c_mul(cb[(int64_t)p * inner + t], lds[t * PS + p]);
        }
    }
    __syncthreads();
    fft_lds<N, T, NT, 1, 0, N>(lds, PS, twl);
    for (int e = threadIdx.x; e < m * T; e += NT) {
        const int t = e % T, p = e / T;
        if (i0 + t < inner) base[(int64_t)p * inner + t] = lds[t * PS + p];
    }
}

// Counts' box of the last pass: row r of the counts (leading indices over M)
// lies at its place over the extents E of the buffer.
struct ConvRows {
    int nlead;
    int M[3];
    int E[3];
    int Mlast;
    int64_t rows;     // prod of the leading M
    int64_t stride;   // values of one entry
};

// Entry blockIdx.y: partial[y * gridDim.x + x] = sum over the rows of block x of
// counts times the inverse transform.  C (d = 1, no axis-0 pass): product here.
template <int N, int NT, int ROWS>
__global__ __launch_bounds__(NT) void k_c2r_dot(const double2* __restrict__ K, const double2* __restrict__ C,
                                                const int64_t* __restrict__ counts, ConvRows cr,
                                                double* __restrict__ partial, const double2* __restrict__ tw) {
    constexpr int H = N / 2, Q = H + 1;
    constexpr int PS = H + 1;
    __shared__ double2 buf[ROWS * PS];
    __shared__ double2 twl[N];
    __shared__ int64_t rsrc[ROWS];
    __shared__ double scratch[NT / 64];
    TwiddleCopy<N, NT> twc;
    twc.fetch(tw);
    const int64_t r0 = (int64_t)blockIdx.x * ROWS;
    const double2* in = K + (int64_t)blockIdx.y * cr.stride;
    for (int rr = threadIdx.x; rr < ROWS; rr += NT) {
        int64_t src = -1;
        if (r0 + rr < cr.rows) {
            uint32_t rem = (uint32_t)(r0 + rr), o = 0, mul = 1;
            for (int k = cr.nlead - 1; k >= 0; --k) {
                o += (rem % (uint32_t)cr.M[k]) * mul;
                rem /= (uint32_t)cr.M[k];
                mul *= (uint32_t)cr.E[k];
            }
            src = o;
        }
        rsrc[rr] = src;
    }
    __syncthreads();
    constexpr int PE = (ROWS * Q + NT - 1) / NT;
#pragma unroll
    for (int u = 0; u < PE; ++u) {
        const int e = threadIdx.x + u * NT;
        if ((ROWS * Q) % NT == 0 || e < ROWS * Q) {
            const int rr = e / Q, k = e - rr * Q;
            double2 v = make_double2(0.0, 0.0);
            if (rsrc[rr] >= 0) v = in[rsrc[rr] * Q + k];
            if (C && rsrc[rr] >= 0) v = c_mul(C[k], v);
            buf[rr * PS + k] = v;
        }
    }
    twc.store(twl, tw);
    __syncthreads();
    constexpr int PER = (ROWS * H + NT - 1) / NT;
    double2 z[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = threadIdx.x + u * NT;
        if (e < ROWS * H) {
            const int rr = e / H, k = e - rr * H;
            const double2 xk = buf[rr * PS + k];
            const double2 xc = c_conj(buf[rr * PS + H - k]);
            const double2 E = c_scale(c_add(xk, xc), 0.5);
            const double2 O = c_scale(c_mulc(c_sub(xk, xc), twl[k]), 0.5);
            z[u] = c_add(E, c_rot<1>(O));
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = threadIdx.x + u * NT;
        if (e < ROWS * H) {
            const int rr = e / H, k = e - rr * H;
            buf[rr * PS + k] = z[u];
        }
    }
    __syncthreads();
    fft_lds<H, ROWS, NT, 1, 0, N>(buf, PS, twl);
    const double quantum = 9.094947017729282379150390625e-13;  // 2^-40
    double acc = 0.0;
    for (int e = threadIdx.x; e < ROWS * H; e += NT) {
        const int rr = e / H, p = 2 * (e - rr * H);
        if (r0 + rr >= cr.rows || p >= cr.Mlast) continue;
        const double2 v = c_scale(buf[rr * PS + p / 2], 2.0);
        const int64_t* c = counts + (r0 + rr) * cr.Mlast + p;
        acc += ((double)c[0] * quantum) * v.x;
        if (p + 1 < cr.Mlast) acc += ((double)c[1] * quantum) * v.y;
    }
    double a[1] = {acc}, out[1];
    block_sum<1, NT>(a, scratch, out);
    if (threadIdx.x == 0) partial[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = out[0];
}

// out[y] = scale * sum of the nblk partial sums of entry y, fixed order.
__global__ __launch_bounds__(256) void k_conv_sum(const double* __restrict__ partial, int nblk, double scale,
                                                  double* __restrict__ out) {
    __shared__ double scratch[4];
    const double* p = partial + (int64_t)blockIdx.x * nblk;
    double acc = 0.0;
#pragma unroll 4
    for (int b = threadIdx.x; b < nblk; b += 256) acc += p[b];
    double v[1] = {acc}, o[1];
    block_sum<1, 256>(v, scratch, o);
    if (threadIdx.x == 0) out[blockIdx.x] = o[0] * scale;
}

// ------------------------------------------------------------------ launchers
// Rows per block of the last pass: one row, or for short rows ~2048 values.
template <int N>
constexpr int conv_rows() { return N >= 256 ? 1 : 2048 / N; }
static int conv_rows_of(int N) { return N >= 256 ? 1 : 2048 / N; }

int conv_blocks(const kdefft_grid& g) {
    int64_t rows = 1;
    for (int k = 0; k + 1 < g.d; ++k) rows *= g.M[k];
    const int r = conv_rows_of(g.P[g.d - 1]);
    return (int)((rows + r - 1) / r);
}

template <int N>
static hipError_t run_conv_axis0(double2* K, const double2* C, int64_t inner, int mk, int m, int nent,
                                 const double2* tw, hipStream_t s) {
    // wide tiles (64 to 128 contiguous bytes per row) once they fill the chip
    constexpr int T = conv_cols<N>();
    if (nent * ((inner + T - 1) / T) >= 256)
        hipLaunchKernelGGL((k_conv_axis0<N, 256, T>), dim3((unsigned)((inner + T - 1) / T), nent), dim3(256), 0, s, K,
                           C, inner, mk, m, tw);
    else
        hipLaunchKernelGGL((k_conv_axis0<N, 256, 1>), dim3((unsigned)inner, nent), dim3(256), 0, s, K, C, inner, mk,
                           m, tw);
    return hipGetLastError();
}

template <int N>
static hipError_t run_c2r_dot(const double2* K, const double2* C, const int64_t* counts, const ConvRows& cr, int nblk,
                              int nent, double* partial, const double2* tw, hipStream_t s) {
    hipLaunchKernelGGL((k_c2r_dot<N, 256, conv_rows<N>()>), dim3((unsigned)nblk, nent), dim3(256), 0, s, K, C, counts,
                       cr, partial, tw);
    return hipGetLastError();
}

#define CONV_SWITCH(NN, CALL)                \
    switch (NN) {                            \
        case 4: return CALL(4);              \
        case 8: return CALL(8);              \
        case 16: return CALL(16);            \
        case 32: return CALL(32);            \
        case 64: return CALL(64);            \
        case 128: return CALL(128);          \
        case 256: return CALL(256);          \
        case 512: return CALL(512);          \
        case 1024: return CALL(1024);        \
        case 2048: return CALL(2048);        \
        case 4096: return CALL(4096);        \
        default: return hipErrorInvalidValue; \
    }

static hipError_t conv_axis0(double2* K, const double2* C, int N, int64_t inner, int mk, int m, int nent,
                             const double2* tw, hipStream_t s) {
#define CALL(NN) run_conv_axis0<NN>(K, C, inner, mk, m, nent, tw, s)
    CONV_SWITCH(N, CALL)
#undef CALL
}
static hipError_t c2r_dot(const double2* K, const double2* C, const int64_t* counts, const ConvRows& cr, int N,
                          int nblk, int nent, double* partial, const double2* tw, hipStream_t s) {
#define CALL(NN) run_c2r_dot<NN>(K, C, counts, cr, nblk, nent, partial, tw, s)
    CONV_SWITCH(N, CALL)
#undef CALL
}

hipError_t conv_sums(const kdefft_grid& g, int mk, int nent, double* kreal, double2* K, const double2* C,
                     const int64_t* counts, double* partial, double scale, double* out, hipStream_t s) {
    const double2* tw;
    hipError_t e = twiddles(&tw);
    if (e != hipSuccess) return e;
    const int d = g.d, m = d > 1 ? g.M[0] : 1;
    e = fft_slices_forward(kreal, K, g, (int64_t)nent * m, s);
    int64_t inner = g.P[d - 1] / 2 + 1;
    for (int k = 1; k + 1 < d; ++k) inner *= g.P[k];
    if (e == hipSuccess && d > 1) e = conv_axis0(K, C, g.P[0], inner, mk, m, nent, tw, s);
    if (e == hipSuccess) e = fft_slices_inverse(K, g, (int64_t)nent * m, s);
    if (e != hipSuccess) return e;
    ConvRows cr{d - 1, {1, 1, 1}, {1, 1, 1}, g.M[d - 1], 1, (int64_t)m * inner};
    for (int k = 0; k + 1 < d; ++k) {
        cr.M[k] = g.M[k];
        cr.E[k] = k == 0 ? m : g.P[k];
        cr.rows *= g.M[k];
    }
    const int nblk = conv_blocks(g);
    e = c2r_dot(K, d == 1 ? C : nullptr, counts, cr, g.P[d - 1], nblk, nent, partial, tw, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_conv_sum, dim3(nent), dim3(256), 0, s, partial, nblk, scale, out);
    return hipGetLastError();
}

}  // namespace kdefft
