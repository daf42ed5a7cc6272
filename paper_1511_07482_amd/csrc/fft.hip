// Multi-dimensional real FFT for the zero-padded grids (Sec. 4, Eq. (19)-(23)):
// LDS-staged Stockham passes along one axis at a time.
//
//  * last axis (contiguous): real-to-complex through a half-length complex
//    transform of the even/odd pairs plus the standard split step, and the
//    inverse complex-to-real;
//  * leading axes (strided): each block loads a tile of T adjacent columns for
//    the full axis length (T * 16 contiguous bytes per row: coalesced), runs T
//    pencils in LDS and writes the tile back in place.  The axis-0 pass of the
//    count transform also forms |C|^2 and transforms it forward again while the
//    tile is still in LDS.
//
// Transforms are unnormalised: forward uses e^{-2 pi i jk/N}, inverse e^{+...}.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "dev_common.h"
#include "internal.h"

namespace kdefft {

// ------------------------------------------------------------------ twiddles
// One table per device; kernels receive its device address as an argument.
// [0, TWN): e^{-2 pi i m / TWN}; then, at offset TWN + N for each power of two
// N <= TWN, the N-point subset e^{-2 pi i j / N}, j < N (the same values, stored
// contiguously so a block can copy the subset it needs in whole cache lines).
static __device__ double2 g_twiddle[3 * TWN];

hipError_t twiddles(const double2** out) {
    static std::mutex mu;
    static const double2* ptr[64] = {nullptr};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!ptr[dev]) {
        // cos/sin of 2 pi m / TWN from the first octant in long double, so that
        // symmetric entries are exactly symmetric and each value is rounded once.
        static double2 host[3 * TWN];
        const long double pi = 3.141592653589793238462643383279502884L;
        for (int m = 0; m < TWN; ++m) {
            int q = m / (TWN / 4), rr = m % (TWN / 4);  // quadrant, remainder
            long double cs, sn;
            if (rr <= TWN / 8) {
                long double a = 2.0L * pi * rr / TWN;
                cs = cosl(a);
                sn = sinl(a);
            } else {
                long double a = 2.0L * pi * (TWN / 4 - rr) / TWN;
                cs = sinl(a);
                sn = cosl(a);
            }
            long double c2, s2;  // rotate by q quarter turns
            switch (q) {
                case 0: c2 = cs; s2 = sn; break;
                case 1: c2 = -sn; s2 = cs; break;
                case 2: c2 = -cs; s2 = -sn; break;
                default: c2 = sn; s2 = -cs; break;
            }
            host[m] = make_double2((double)c2, -(double)s2);  // e^{-i theta}
        }
        for (int N = 1; N <= TWN; N *= 2)
            for (int j = 0; j < N; ++j) host[TWN + N + j] = host[j * (TWN / N)];
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_twiddle), host, sizeof(host), 0, hipMemcpyHostToDevice);
        if (e != hipSuccess) return e;
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_twiddle));
        if (e != hipSuccess) return e;
        ptr[dev] = static_cast<const double2*>(p);
    }
    *out = ptr[dev];
    return hipSuccess;
}

// ------------------------------------------------------------------ last axis
// Optional input maps of the last-axis passes.
//  * CountSrc: the R2C input row is read straight from the int64 grid counts,
//    or gathered from the binning's corner slots (c = count 2^-40 at [0, M)^d
//    of the circular layout, zero elsewhere), so the zero-padded real array is
//    never materialised.  The launch covers the rows inside the counts' box:
//    row r is the counts' row r (leading indices over M), stored at its place in
//    the padded grid; the padding's zero rows are not written (the next pass
//    never reads them).
//  * RowFlip: the C2R pass writes input row l (l_0 in [0, P_0/2] only) to
//    output row -l, and, as the real output f is even, f(l) = f(-l), that row
//    reversed to output row l.
struct CountSrc {
    const int64_t* counts;  // nullptr: read the real input array
    int d;
    int M[4];
    int P[4];
    int slots;              // counts holds the binning's corner slots, gathered here
    int64_t* sum_out;       // the gathered counts, written when slots is set
    int32_t* reach;         // if set, receives M - 1 per axis (block 0)
};

// The corner slots' part of the count at position p of a row (base: the cell of
// its first position; bit j - 1 of lmask: the row's index along axis d-1-j is
// >= 1).  The count of cell i is the sum over s of slot s of the record of cell
// i - e(s), e(s) = the sum over the set bits j of s of the stride of axis d-1-j,
// for the slots whose lower cell exists.  Slots 2t and 2t + 1 of a record are
// 16 bytes: x collects the even slots, which belong to position p, y the odd
// ones, which belong to p + 1.  Exact (unsigned 64-bit sums).
template <int NSA>
__device__ __forceinline__ ulonglong2 gather_slots(const int64_t* __restrict__ slots, int64_t base, int p, int lmask,
                                                   const int* M, int d) {
    constexpr int NP = 1 << (NSA - 1);
    const ulonglong2* rec = reinterpret_cast<const ulonglong2*>(slots);
    const int64_t st1 = NSA > 1 ? M[d - 1] : 0;
    const int64_t st2 = NSA > 2 ? st1 * M[d - 2] : 0;
    ulonglong2 sum = make_ulonglong2(0, 0);
#pragma unroll
    for (int t = 0; t < NP; ++t) {
        if ((t & 1 && !(lmask & 1)) || (t & 2 && !(lmask & 2))) continue;
        const ulonglong2 v = rec[(base + p - (t & 1 ? st1 : 0) - (t & 2 ? st2 : 0)) * NP + t];
        sum.x += v.x;
        sum.y += v.y;
    }
    return sum;
}

struct RowFlip {
    int on;
    int nlead;
    int P[3];
    int mlast;   // > 0: positions with |lag| > M - 1 along any axis are written as exact zeros (M of the
    int M[3];    // last axis: mlast, of the leading ones: M); rows of zeros are not read
};

// Output row -l of source row l (each leading index negated modulo P); zero:
// both are rows of zeros; inner: 0 < l_0 < P_0 / 2, so that row l is not
// itself read.  Row indices of the passes are below 2^31 (checked on the
// host), so rows are decoded with 32-bit divisions.
__device__ __forceinline__ int64_t flip_row(int64_t row, const RowFlip& f, bool& zero, bool& inner) {
    uint32_t r = (uint32_t)row, out = 0, mul = 1;
    zero = false;
    inner = false;
    for (int k = f.nlead - 1; k >= 0; --k) {
        const uint32_t p = (uint32_t)f.P[k], i = r % p;
        r /= p;
        if (f.mlast > 0 && i >= (uint32_t)f.M[k] && i <= p - (uint32_t)f.M[k]) zero = true;
        out += (i == 0 ? 0u : p - i) * mul;
        mul *= p;
        if (k == 0) inner = i > 0 && i < p / 2;
    }
    return out;
}

// Rows per block for a last-axis pass of real length N.
template <int N>
constexpr int last_rows() { return (N / 2) >= 2048 ? 1 : 2048 / (N / 2); }

template <int N, int NT, int ROWS, int RADIX>
__global__ __launch_bounds__(NT) void k_r2c_last(const double* __restrict__ in, double2* __restrict__ out,
                                                 int64_t rows, const double2* __restrict__ tw, CountSrc cs) {
    constexpr int H = N / 2, Q = H + 1;
    constexpr int PS = H + 1;
    __shared__ double2 buf[ROWS * PS];
    __shared__ double2 twl[N];
    TwiddleCopy<N, NT> twc;
    twc.fetch(tw);
    const int64_t r0 = (int64_t)blockIdx.x * ROWS;
    const double2* src = reinterpret_cast<const double2*>(in);
    if (cs.reach && blockIdx.x == 0 && threadIdx.x < (unsigned)cs.d) cs.reach[threadIdx.x] = cs.M[threadIdx.x] - 1;
    if (cs.counts) {
        const double quantum = 9.094947017729282379150390625e-13;  // 2^-40
        const int Ml = cs.M[cs.d - 1];
        // offset of each row's counts (-1: past the end), decoded once per row
        __shared__ int64_t rbase[ROWS];
        __shared__ int rmask[ROWS];   // bit 0: the row's index along axis d-2 is >= 1; bit 1: along d-3
        for (int rr = threadIdx.x; rr < ROWS; rr += NT) {
            const int64_t row = r0 + rr;
            uint32_t rem = (uint32_t)row;
            int mask = 0;
            for (int k = cs.d - 2; k >= 0 && k >= cs.d - 3; --k) {
                const uint32_t m = (uint32_t)cs.M[k];
                if (rem % m >= 1) mask |= k == cs.d - 2 ? 1 : 2;
                rem /= m;
            }
            rbase[rr] = row < rows ? row * Ml : -1;
            rmask[rr] = mask;
        }
        __syncthreads();
        constexpr int PE = (ROWS * H + NT - 1) / NT;
        double2 v[PE];
        if (cs.slots) {
            // Each 16-byte piece is read once, by one lane; the odd slots reach
            // their cell through LDS.  Reading the 2^d slots of each cell, 8 bytes
            // each, was bound by the lines per load instruction: d = 4, M = 32
            // 42 -> 30 us, d = 3, M = 64 14.7 -> 9.6 us.
            uint64_t* part = reinterpret_cast<uint64_t*>(buf);   // rows of 2 PS words
            const int lw = Ml <= H ? ilog2c(H) : ilog2c(N);      // lanes per row: the positions that can hold counts
            uint64_t odd[2 * PE];
#pragma unroll
            for (int u = 0; u < 2 * PE; ++u) {
                odd[u] = 0;
                const int e = threadIdx.x + u * NT, rr = e >> lw, p = e - (rr << lw);
                if (rr < ROWS && p < Ml && rbase[rr] >= 0) {
                    const int64_t base = rbase[rr];
                    const int lm = rmask[rr];
                    const ulonglong2 t = cs.d == 1   ? gather_slots<1>(cs.counts, base, p, lm, cs.M, cs.d)
                                         : cs.d == 2 ? gather_slots<2>(cs.counts, base, p, lm, cs.M, cs.d)
                                                     : gather_slots<3>(cs.counts, base, p, lm, cs.M, cs.d);
                    part[rr * 2 * PS + p] = t.x;
                    odd[u] = t.y;
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2 * PE; ++u) {
                const int e = threadIdx.x + u * NT, rr = e >> lw, p = e - (rr << lw);
                if (rr < ROWS && p + 1 < Ml && rbase[rr] >= 0) part[rr * 2 * PS + p + 1] += odd[u];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PE; ++u) {
                const int e = threadIdx.x + u * NT;
                v[u] = make_double2(0.0, 0.0);
                if ((ROWS * H) % NT == 0 || e < ROWS * H) {
                    const int rr = e / H, p = 2 * (e - rr * H);
                    const int64_t base = rbase[rr];
                    const uint64_t* c = part + rr * 2 * PS + p;
                    if (base >= 0 && p < Ml) {
                        cs.sum_out[base + p] = (int64_t)c[0];
                        v[u].x = (double)(int64_t)c[0] * quantum;
                    }
                    if (base >= 0 && p + 1 < Ml) {
                        cs.sum_out[base + p + 1] = (int64_t)c[1];
                        v[u].y = (double)(int64_t)c[1] * quantum;
                    }
                }
            }
            __syncthreads();
        } else {
#pragma unroll
            for (int u = 0; u < PE; ++u) {
                const int e = threadIdx.x + u * NT;
                v[u] = make_double2(0.0, 0.0);
                if ((ROWS * H) % NT == 0 || e < ROWS * H) {
                    const int rr = e / H, p = 2 * (e - rr * H);
                    const int64_t base = rbase[rr];
                    if (base >= 0 && p < Ml) v[u].x = (double)cs.counts[base + p] * quantum;
                    if (base >= 0 && p + 1 < Ml) v[u].y = (double)cs.counts[base + p + 1] * quantum;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < PE; ++u) {
            const int e = threadIdx.x + u * NT;
            if ((ROWS * H) % NT == 0 || e < ROWS * H) {
                const int rr = e / H, m = e - rr * H;
                buf[rr * PS + m] = v[u];
            }
        }
    } else {
        constexpr int PE = (ROWS * H + NT - 1) / NT;
#pragma unroll
        for (int u = 0; u < PE; ++u) {
            const int e = threadIdx.x + u * NT;
            if ((ROWS * H) % NT == 0 || e < ROWS * H) {
                const int rr = e / H, m = e - rr * H;
                const int64_t row = r0 + rr;
                buf[rr * PS + m] = row < rows ? src[row * H + m] : make_double2(0.0, 0.0);
            }
        }
    }
    twc.store(twl, tw);
    __syncthreads();
    fft_lds<H, ROWS, NT, -1, RADIX, N>(buf, PS, twl);
    __shared__ int64_t rout[ROWS];   // output row of each row: its place in the padded grid when pruned
    for (int rr = threadIdx.x; rr < ROWS; rr += NT) {
        int64_t row = r0 + rr;
        if (cs.counts) {
            uint32_t rem = (uint32_t)row, o = 0, mul = 1;
            for (int k = cs.d - 2; k >= 0; --k) {
                const uint32_t m = (uint32_t)cs.M[k];
                o += (rem % m) * mul;
                rem /= m;
                mul *= (uint32_t)cs.P[k];
            }
            row = o;
        }
        rout[rr] = row;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < ROWS * Q; e += NT) {
        const int rr = e / Q, k = e - rr * Q;
        if (r0 + rr >= rows) continue;
        const int64_t row = rout[rr];
        const double2 zk = buf[rr * PS + (k == H ? 0 : k)];
        const double2 zc = c_conj(buf[rr * PS + (k == 0 ? 0 : H - k)]);
        const double2 E = c_scale(c_add(zk, zc), 0.5);
        const double2 O = c_rot<-1>(c_scale(c_sub(zk, zc), 0.5));  // (zk - zc)/(2i)
        const double2 w = twl[k];
        out[row * Q + k] = c_add(E, c_mul(w, O));
    }
}

template <int N, int NT, int ROWS, int RADIX>
__global__ __launch_bounds__(NT) void k_c2r_last(const double2* __restrict__ in, double* __restrict__ out,
                                                 int64_t rows, const double2* __restrict__ tw, RowFlip fl) {
    constexpr int H = N / 2, Q = H + 1;
    constexpr int PS = H + 1;
    __shared__ double2 buf[ROWS * PS];
    __shared__ double2 twl[N];
    // source row (-1: past the end or zeros) and destination rows (-1: none), decoded once per row
    __shared__ int64_t rsrc[ROWS], rdst[ROWS], rmir[ROWS];
    TwiddleCopy<N, NT> twc;
    twc.fetch(tw);
    const int64_t r0 = (int64_t)blockIdx.x * ROWS;
    for (int rr = threadIdx.x; rr < ROWS; rr += NT) {
        const int64_t row = r0 + rr;
        bool zero = false, inner = false;
        const int64_t dst = fl.on ? flip_row(row, fl, zero, inner) : row;
        rsrc[rr] = row < rows && !zero ? row : -1;
        rdst[rr] = row < rows ? dst : -1;
        rmir[rr] = row < rows && inner ? row : -1;
    }
    __syncthreads();
    {
        constexpr int PE = (ROWS * Q + NT - 1) / NT;   // unrolled: the loads in flight together
#pragma unroll
        for (int u = 0; u < PE; ++u) {
            const int e = threadIdx.x + u * NT;
            if ((ROWS * Q) % NT == 0 || e < ROWS * Q) {
                const int rr = e / Q, k = e - rr * Q;
                const int64_t src_row = rsrc[rr];
                buf[rr * PS + k] = src_row >= 0 ? in[src_row * Q + k] : make_double2(0.0, 0.0);
            }
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
            const double2 O = c_scale(c_mulc(c_sub(xk, xc), twl[k]), 0.5);  // * e^{+i..}
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
    fft_lds<H, ROWS, NT, 1, RADIX, N>(buf, PS, twl);
    double2* dst = reinterpret_cast<double2*>(out);
    for (int e = threadIdx.x; e < ROWS * H; e += NT) {
        const int rr = e / H, m = e - rr * H;
        const int64_t row = rdst[rr], mir = rmir[rr];
        if (row < 0) continue;
        double2 v = c_scale(buf[rr * PS + m], 2.0);
        // positions -2m and -2m - 1 (modulo N) of the row
        double2 w = make_double2(2.0 * buf[rr * PS + (m == 0 ? 0 : H - m)].x, 2.0 * buf[rr * PS + H - 1 - m].y);
        if (fl.mlast > 0) {
            // positions 2m, 2m + 1 hold lags p (p < N/2) or p - N
            const int p0 = 2 * m, p1 = 2 * m + 1;
            if (p0 > fl.mlast - 1 && p0 < N - (fl.mlast - 1)) v.x = w.x = 0.0;
            if (p1 > fl.mlast - 1 && p1 < N - (fl.mlast - 1)) v.y = w.y = 0.0;
        }
        dst[row * H + m] = v;
        if (mir >= 0) dst[mir * H + m] = w;
    }
}

// ------------------------------------------------------------------ strided axes
// Columns per tile: the largest power of two <= 16 whose padded tile fits 64 KiB.
template <int N>
constexpr int tile_cols() {
    return 4096 / (N + 1) >= 16 ? 16 : 4096 / (N + 1) >= 8 ? 8 : 4096 / (N + 1) >= 4 ? 4
         : 4096 / (N + 1) >= 2 ? 2 : 1;
}

// Zero structure of a forward count-transform pass along axis a (pruning):
// the counts fill [0, M)^d of the padded P^d grid, so before the pass a
// column (outer index i_0..i_{a-1} over the axes before a) can be nonzero only
// if every i_k < M_k, and within it only its first M_a entries.  The launch
// covers the live columns only (its outer index runs over the M_k extents and
// is placed in the P_k-extent buffer; the dead columns are neither read nor
// written: the next pass, along a - 1, reads only live columns' outputs), and
// only the first nlive entries of a column are read.  na = 0, nlive = N: the
// dense transform.
struct Prune {
    int na;       // axes before the pass's axis
    int P[3];     // their extents (outer index digits, major first)
    int M[3];     // their count extents
    int nlive;    // entries of a live column that can be nonzero
    int nstore;   // entries of a column that are stored (0: all)
    int nstore2;  // MODE 1: entries of a column of out2 that are stored (0: all)
    uint32_t blocks = 0;   // tiles of the launch (set there)
};

// MODE 0: in-place transform.  MODE 1: forward transform stored in place
// (the finished count spectrum C), then |C|^2 transformed forward again and
// stored to out2.  MODE 2: the last forward pass of |C|^2 along the leading
// axes: that transform W of real values is Hermitian, W(-l) = conj W(l) over
// the leading indices, so the launch visits the columns with l_0 in [0, P_0/2]
// (na the axes before the pass's, M_0 = P_0/2 + 1) and stores those with 0 <
// l_0 < P_0/2 at -l too.  The passes stream at the rate of a copy, so the bytes
// they skip are the gain: d = 4, P = 64 (138 MB a spectrum), transform and
// autocorrelation 309 us with every column transformed and read, 221 so.
template <int N, int NT, int DIR, int MODE, int T, int RADIX>
__global__ __launch_bounds__(NT) void k_c2c_strided(double2* __restrict__ buf, double2* __restrict__ out2,
                                                    int64_t inner, int64_t tiles,
                                                    const double2* __restrict__ tw, Prune pr) {
    constexpr int PS = T > 1 ? N + 1 : N;
    __shared__ double2 lds[T * PS];
    __shared__ double2 twl[N];
    TwiddleCopy<N, NT> twc;
    twc.fetch(tw);
    // Narrow tiles share cache lines with their neighbours, and consecutive
    // blocks run on different XCDs (of 8, each with its own L2): deal each XCD a
    // contiguous range of tiles instead (d = 2, P = 512, 257 single columns: 10.3
    // -> 7.6 us; d = 3, P = 256, 8 columns: whole transform 222 -> 187; tiles of 16
    // columns gain nothing).  The grid is then a multiple
    // of 8.
    uint32_t bid = blockIdx.x;
    if constexpr (T <= 8) {
        bid = (bid % 8) * (gridDim.x / 8) + bid / 8;
        if (bid >= pr.blocks) return;
    }
    // block indices and outer indices are below 2^32: 32-bit divisions
    const uint32_t ol = bid / (uint32_t)tiles;
    uint32_t o = ol, om = 0;   // om: -o
    bool mirror = false;
    if (pr.na > 0) {   // live column ol (extents M) -> its outer index in the buffer (extents P)
        uint32_t rem = ol, mul = 1;
        o = 0;
        for (int k = pr.na - 1; k >= 0; --k) {
            const uint32_t m = (uint32_t)pr.M[k], p = (uint32_t)pr.P[k], i = rem % m;
            o += i * mul;
            om += (i == 0 ? 0u : p - i) * mul;
            rem /= m;
            mul *= p;
            if (k == 0) mirror = i > 0 && i < p / 2;
        }
    }
    const int64_t i0 = (int64_t)(bid - ol * (uint32_t)tiles) * T;
    double2* base = buf + (int64_t)o * N * inner + i0;
    {
        constexpr int PE = (N * T + NT - 1) / NT;   // unrolled: the loads in flight together
#pragma unroll
        for (int u = 0; u < PE; ++u) {
            const int e = threadIdx.x + u * NT;
            if ((N * T) % NT == 0 || e < N * T) {
                const int t = e % T, p = e / T;
                lds[t * PS + p] =
                    (i0 + t < inner && p < pr.nlive) ? base[(int64_t)p * inner + t] : make_double2(0.0, 0.0);
            }
        }
    }
    twc.store(twl, tw);
    __syncthreads();
    fft_lds<N, T, NT, DIR, RADIX, N>(lds, PS, twl);
    for (int e = threadIdx.x; e < N * T; e += NT) {
        const int t = e % T, p = e / T;
        if (i0 + t < inner && p < pr.nstore) base[(int64_t)p * inner + t] = lds[t * PS + p];
    }
    if constexpr (MODE == 2) {
        if (mirror) {
            double2* b2 = buf + (int64_t)om * N * inner + i0;
            for (int e = threadIdx.x; e < N * T; e += NT) {
                const int t = e % T, p = e / T;
                if (i0 + t < inner) b2[(int64_t)p * inner + t] = c_conj(lds[t * PS + (p == 0 ? 0 : N - p)]);
            }
        }
    }
    if constexpr (MODE == 1) {
        for (int e = threadIdx.x; e < N * T; e += NT) {
            const int t = e % T, p = e / T;
            const double2 v = lds[t * PS + p];
            lds[t * PS + p] = make_double2(v.x * v.x + v.y * v.y, 0.0);
        }
        __syncthreads();
        fft_lds<N, T, NT, -1, RADIX, N>(lds, PS, twl);
        double2* b2 = out2 + (int64_t)o * N * inner + i0;
        for (int e = threadIdx.x; e < N * T; e += NT) {
            const int t = e % T, p = e / T;
            if (i0 + t < inner && p < pr.nstore2) b2[(int64_t)p * inner + t] = lds[t * PS + p];
        }
    }
}

// |C|^2 for d = 1 (no leading axis).
__global__ void k_abs2(const double2* __restrict__ in, double2* __restrict__ out, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double2 v = in[i];
        out[i] = make_double2(v.x * v.x + v.y * v.y, 0.0);
    }
}

// ------------------------------------------------------------------ dispatch
static int ilog2i(int n) { int k = 0; while ((1 << k) < n) ++k; return k; }

// Launch shapes.  Default: ~2048 complex values per block (256 threads).
// Small problems (fewer than ~512 blocks at the default shape) take one or a
// few pencils per block instead, so more CUs take part: the pencils of one
// wavefront's shape on 256 threads, whose extra lanes shorten the loads and
// stores that bound these passes (part of them idle in the stages).
constexpr int64_t kMinBlocks = 512;

// pencils of one wavefront (at most 16, ~512 values), and half of them (at
// least one) for the 256-thread small shape
template <int N>
constexpr int small_rows() { return (N / 2) >= 512 ? 1 : ((512 / (N / 2)) > 16 ? 16 : 512 / (N / 2)); }
template <int N>
constexpr int deep_rows() { return small_rows<N>() > 1 ? small_rows<N>() / 2 : 1; }

// FFT-stage schedules (the tuner's choices, per grid shape):
//   FS_AUTO    the shape rule above, radix-8 stages first;
//   FS_RADIX4  the same shapes, radix-4 stages (one radix-8 or 2 when log2 is odd);
//   FS_WIDE    256-thread blocks of the default shape for every pass;
//   FS_NARROW  one-wavefront blocks for every pass that has them;
//   FS_HALF    strided passes on T/2-column tiles (twice the blocks), last axis as FS_AUTO;
//   FS_DEEP    the small problems' 256-thread shapes for every pass that has them.
enum { FS_AUTO = 0, FS_RADIX4 = 1, FS_WIDE = 2, FS_NARROW = 3, FS_HALF = 4, FS_DEEP = 5 };

// Radix-4 stages for schedule FS_RADIX4, and under the default schedule for
// 64-point passes (4 x 4 x 4 measured up to 6% faster than 8 x 8 over a
// d = 4, P = 64 transform streaming from HBM; other lengths keep radix 8 first).
template <int N>
constexpr bool radix4_for_default() { return N == 64; }
template <int N>
static bool radix4_for(int fs) { return fs == FS_RADIX4 || (fs == FS_AUTO && radix4_for_default<N>()); }

// Last-axis launch shapes: ROWS rows on 256 threads, small_rows on one
// wavefront, deep_rows on 256 threads.
enum { SH_WIDE = 0, SH_NARROW = 1, SH_DEEP = 2 };

template <int N, int RADIX>
static void launch_r2c_shape(int sh, const double* in, double2* out, int64_t rows, const double2* tw,
                             hipStream_t s, CountSrc cs) {
    constexpr int ROWS = last_rows<N>();
    constexpr int RS = small_rows<N>();
    constexpr int RD = deep_rows<N>();
    if (sh == SH_NARROW && RS < ROWS)
        hipLaunchKernelGGL((k_r2c_last<N, 64, RS, RADIX>), dim3((unsigned)((rows + RS - 1) / RS)), dim3(64), 0, s,
                           in, out, rows, tw, cs);
    else if (sh == SH_DEEP && RS < ROWS)
        hipLaunchKernelGGL((k_r2c_last<N, 256, RD, RADIX>), dim3((unsigned)((rows + RD - 1) / RD)), dim3(256), 0,
                           s, in, out, rows, tw, cs);
    else
        hipLaunchKernelGGL((k_r2c_last<N, 256, ROWS, RADIX>), dim3((unsigned)((rows + ROWS - 1) / ROWS)), dim3(256),
                           0, s, in, out, rows, tw, cs);
}

template <int N, int RADIX>
static void launch_c2r_shape(int sh, const double2* in, double* out, int64_t rows, const double2* tw,
                             hipStream_t s, RowFlip fl) {
    constexpr int ROWS = last_rows<N>();
    constexpr int RS = small_rows<N>();
    constexpr int RD = deep_rows<N>();
    if (sh == SH_NARROW && RS < ROWS)
        hipLaunchKernelGGL((k_c2r_last<N, 64, RS, RADIX>), dim3((unsigned)((rows + RS - 1) / RS)), dim3(64), 0, s,
                           in, out, rows, tw, fl);
    else if (sh == SH_DEEP && RS < ROWS)
        hipLaunchKernelGGL((k_c2r_last<N, 256, RD, RADIX>), dim3((unsigned)((rows + RD - 1) / RD)), dim3(256), 0,
                           s, in, out, rows, tw, fl);
    else
        hipLaunchKernelGGL((k_c2r_last<N, 256, ROWS, RADIX>), dim3((unsigned)((rows + ROWS - 1) / ROWS)), dim3(256),
                           0, s, in, out, rows, tw, fl);
}

// last-axis launch shape for schedule fs
template <int N>
static int last_shape(int64_t rows, int fs) {
    constexpr int ROWS = last_rows<N>();
    if (fs == FS_WIDE) return SH_WIDE;
    if (fs == FS_NARROW) return SH_NARROW;
    if (fs == FS_DEEP) return SH_DEEP;
    return (rows + ROWS - 1) / ROWS < kMinBlocks ? SH_DEEP : SH_WIDE;
}

template <int N>
static hipError_t run_r2c_last(const double* in, double2* out, int64_t rows, const double2* tw, hipStream_t s,
                               CountSrc cs, int fs) {
    const int sh = last_shape<N>(rows, fs);
    if (radix4_for<N>(fs))
        launch_r2c_shape<N, 1>(sh, in, out, rows, tw, s, cs);
    else
        launch_r2c_shape<N, 0>(sh, in, out, rows, tw, s, cs);
    return hipGetLastError();
}
template <int N>
static hipError_t run_c2r_last(const double2* in, double* out, int64_t rows, const double2* tw, hipStream_t s,
                               RowFlip fl, int fs) {
    const int sh = last_shape<N>(rows, fs);
    if (radix4_for<N>(fs))
        launch_c2r_shape<N, 1>(sh, in, out, rows, tw, s, fl);
    else
        launch_c2r_shape<N, 0>(sh, in, out, rows, tw, s, fl);
    return hipGetLastError();
}

template <int N, int NT, int T, int RADIX>
static void launch_c2c_t(double2* buf, double2* out2, int64_t outer, int64_t inner, int dir, int mode,
                         const double2* tw, hipStream_t s, Prune pr) {
    const int64_t tiles = (inner + T - 1) / T, blocks = outer * tiles;
    pr.blocks = (uint32_t)blocks;
    const dim3 grid((unsigned)(T <= 8 ? (blocks + 7) / 8 * 8 : blocks));
    if (mode == 1)
        hipLaunchKernelGGL((k_c2c_strided<N, NT, -1, 1, T, RADIX>), grid, dim3(NT), 0, s, buf, out2, inner, tiles,
                           tw, pr);
    else if (mode == 2)
        hipLaunchKernelGGL((k_c2c_strided<N, NT, -1, 2, T, RADIX>), grid, dim3(NT), 0, s, buf, out2, inner, tiles,
                           tw, pr);
    else if (dir < 0)
        hipLaunchKernelGGL((k_c2c_strided<N, NT, -1, 0, T, RADIX>), grid, dim3(NT), 0, s, buf, out2, inner, tiles,
                           tw, pr);
    else
        hipLaunchKernelGGL((k_c2c_strided<N, NT, 1, 0, T, RADIX>), grid, dim3(NT), 0, s, buf, out2, inner, tiles,
                           tw, pr);
}

// Slab tiles: when the axis is the last leading one its inner extent is the
// half-spectrum length Q = P/2 + 1 (17, 33, 65, ...), which T-column tiles
// cover raggedly (33 = 16 + 16 + 1).  For Q = 17 and 33 one block takes the
// whole contiguous [N][Q] slab instead (fully coalesced, no partial tile)
// while it fits 80 KiB of LDS.
template <int N, int Q>
constexpr bool slab_fits() { return N >= 8 && Q * (N + 1) * 16 <= 81920; }

template <int N, int RADIX>
static void run_c2c_r(double2* buf, double2* out2, int64_t outer, int64_t inner, int dir, int mode,
                      const double2* tw, hipStream_t s, int fs, const Prune& pr) {
    constexpr int T = tile_cols<N>();
    constexpr int TS = N >= 64 ? 1 : (64 / N > 16 ? 16 : 64 / N);  // one radix pass per lane
    constexpr int TH = T > 1 ? T / 2 : 1;
    const bool small = outer * ((inner + T - 1) / T) < kMinBlocks;
    if (fs != FS_NARROW && fs != FS_HALF && fs != FS_DEEP) {
        if constexpr (slab_fits<N, 33>()) {
            if (inner == 33 && (outer >= kMinBlocks || fs == FS_WIDE)) {
                launch_c2c_t<N, 256, 33, RADIX>(buf, out2, outer, inner, dir, mode, tw, s, pr);
                return;
            }
        }
        if constexpr (slab_fits<N, 17>()) {
            if (inner == 17 && (outer >= kMinBlocks || fs == FS_WIDE)) {
                launch_c2c_t<N, 256, 17, RADIX>(buf, out2, outer, inner, dir, mode, tw, s, pr);
                return;
            }
        }
    }
    // Four columns (half a cache line) where the full tiles make few blocks and
    // these enough: d = 3, P = 128, passes over 64 or 65 rows of 65 columns, us,
    // single columns -> four: 14.7 -> 6.3 and 28.2 -> 9.1; axis 0 (520 full
    // tiles), transform and autocorrelation 57.2 -> 54.6.
    if constexpr (N >= 64 && T > 4) {
        if (fs != FS_NARROW && fs != FS_HALF && fs != FS_DEEP && fs != FS_WIDE &&
            outer * ((inner + T - 1) / T) < 2 * kMinBlocks && outer * ((inner + 3) / 4) >= kMinBlocks) {
            launch_c2c_t<N, 256, 4, RADIX>(buf, out2, outer, inner, dir, mode, tw, s, pr);
            return;
        }
    }
    if constexpr (TS < T) {
        // one-wavefront blocks (FS_NARROW), or the same tiles on 256 threads
        if (fs == FS_NARROW) {
            launch_c2c_t<N, 64, TS, RADIX>(buf, out2, outer, inner, dir, mode, tw, s, pr);
            return;
        }
        if (fs == FS_DEEP || (fs != FS_WIDE && small)) {
            launch_c2c_t<N, 256, TS, RADIX>(buf, out2, outer, inner, dir, mode, tw, s, pr);
            return;
        }
    }
    if constexpr (RADIX == 0 && TH < T) {
        if (fs == FS_HALF) {
            launch_c2c_t<N, 256, TH, 0>(buf, out2, outer, inner, dir, mode, tw, s, pr);
            return;
        }
    }
    launch_c2c_t<N, 256, T, RADIX>(buf, out2, outer, inner, dir, mode, tw, s, pr);
}

template <int N>
static hipError_t run_c2c(double2* buf, double2* out2, int64_t outer, int64_t inner, int dir, int mode,
                          const double2* tw, hipStream_t s, int fs, const Prune& pr) {
    if (radix4_for<N>(fs))
        run_c2c_r<N, 1>(buf, out2, outer, inner, dir, mode, tw, s, fs, pr);
    else
        run_c2c_r<N, 0>(buf, out2, outer, inner, dir, mode, tw, s, fs, pr);
    return hipGetLastError();
}

#define KDEFFT_SWITCH_N(LOGN, CALL)                           \
    switch (LOGN) {                                          \
        case 1: return CALL(2);                              \
        case 2: return CALL(4);                              \
        case 3: return CALL(8);                              \
        case 4: return CALL(16);                             \
        case 5: return CALL(32);                             \
        case 6: return CALL(64);                             \
        case 7: return CALL(128);                            \
        case 8: return CALL(256);                            \
        case 9: return CALL(512);                            \
        case 10: return CALL(1024);                          \
        case 11: return CALL(2048);                          \
        case 12: return CALL(4096);                          \
        default: return hipErrorInvalidValue;                \
    }

static hipError_t r2c_last(const double* in, double2* out, int64_t rows, int N, const double2* tw, hipStream_t s,
                           CountSrc cs = CountSrc{nullptr, 0, {0, 0, 0, 0}, {0, 0, 0, 0}, 0, nullptr, nullptr},
                           int fs = FS_AUTO) {
#define CALL(NN) run_r2c_last<NN>(in, out, rows, tw, s, cs, fs)
    if (N < 4) return hipErrorInvalidValue;
    KDEFFT_SWITCH_N(ilog2i(N), CALL)
#undef CALL
}
static hipError_t c2r_last(const double2* in, double* out, int64_t rows, int N, const double2* tw, hipStream_t s,
                           RowFlip fl = RowFlip{0, 0, {1, 1, 1}, 0, {1, 1, 1}}, int fs = FS_AUTO) {
#define CALL(NN) run_c2r_last<NN>(in, out, rows, tw, s, fl, fs)
    if (N < 4) return hipErrorInvalidValue;
    KDEFFT_SWITCH_N(ilog2i(N), CALL)
#undef CALL
}
static hipError_t c2c(double2* buf, double2* out2, int64_t outer, int N, int64_t inner, int dir, int mode,
                      const double2* tw, hipStream_t s, int fs = FS_AUTO, Prune pr = Prune{0, {1, 1, 1}, {1, 1, 1}, 0, 0, 0}) {
    if (pr.nlive <= 0 || pr.nlive > N) pr.nlive = N;
    if (pr.nstore <= 0 || pr.nstore > N) pr.nstore = N;
    if (pr.nstore2 <= 0 || pr.nstore2 > N) pr.nstore2 = N;
    if (pr.na > 0) {   // the launch covers the live columns only
        outer = 1;
        for (int k = 0; k < pr.na; ++k) outer *= pr.M[k];
    }
#define CALL(NN) run_c2c<NN>(buf, out2, outer, inner, dir, mode, tw, s, fs, pr)
    KDEFFT_SWITCH_N(ilog2i(N), CALL)
#undef CALL
}

// Shape helpers: the half-spectrum is [P_0, ..., P_{d-2}, Q].
static int64_t lead_count(const kdefft_grid& g) {
    int64_t r = 1;
    for (int k = 0; k + 1 < g.d; ++k) r *= g.P[k];
    return r;
}
// the kernels decode row and column indices in 32 bits
static bool shape_ok(const kdefft_grid& g) {
    return g.d >= 1 && g.d <= 4 && lead_count(g) * (g.P[g.d - 1] / 2 + 1) < (int64_t(1) << 31);
}
static void axis_shape(const kdefft_grid& g, int axis, int64_t* outer, int64_t* inner) {
    int64_t o = 1, in = g.P[g.d - 1] / 2 + 1;
    for (int k = 0; k < axis; ++k) o *= g.P[k];
    for (int k = axis + 1; k + 1 < g.d; ++k) in *= g.P[k];
    *outer = o;
    *inner = in;
}

// Axes d-1..1 of real arrays of `slices` slices along axis 0 (the axis-0 index,
// or several arrays' ones, leads): in [slices, P_1, .., P_{d-1}] -> out
// [slices, P_1, .., Q].
hipError_t fft_slices_forward(const double* in, double2* out, const kdefft_grid& g, int64_t slices, hipStream_t s) {
    if (!shape_ok(g)) return hipErrorInvalidValue;
    const double2* tw;
    hipError_t e = twiddles(&tw);
    if (e != hipSuccess) return e;
    int64_t rows = slices;
    for (int k = 1; k + 1 < g.d; ++k) rows *= g.P[k];
    e = r2c_last(in, out, rows, g.P[g.d - 1], tw, s);
    int64_t inner = g.P[g.d - 1] / 2 + 1;
    for (int ax = g.d - 2; ax >= 1 && e == hipSuccess; --ax) {
        rows /= g.P[ax];
        e = c2c(out, nullptr, rows, g.P[ax], inner, -1, 0, tw, s);
        inner *= g.P[ax];
    }
    return e;
}

// The inverse along axes 1..d-2 in place, for the nodes inside the counts' box:
// of each axis only the entries below M are stored and, along the next one,
// visited.
hipError_t fft_slices_inverse(double2* buf, const kdefft_grid& g, int64_t slices, hipStream_t s) {
    if (!shape_ok(g) || slices >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    const double2* tw;
    hipError_t e = twiddles(&tw);
    if (e != hipSuccess) return e;
    for (int ax = 1; ax + 1 < g.d && e == hipSuccess; ++ax) {
        int64_t inner = g.P[g.d - 1] / 2 + 1;
        for (int k = ax + 1; k + 1 < g.d; ++k) inner *= g.P[k];
        Prune pr{ax, {(int)slices, 1, 1}, {(int)slices, 1, 1}, 0, g.M[ax], 0};
        for (int k = 1; k < ax; ++k) {
            pr.P[k] = g.P[k];
            pr.M[k] = g.M[k];
        }
        e = c2c(buf, nullptr, slices, g.P[ax], inner, 1, 0, tw, s, FS_AUTO, pr);
    }
    return e;
}

// wmix set: as fft_prepare_nd; NULL: the count spectrum alone.
static hipError_t counts_forward(const int64_t* src, int slots, int64_t* counts, double2* spec, double2* wmix,
                                 const kdefft_grid& g, hipStream_t s, int fs, int32_t* reach) {
    if (fs < 0 || fs >= FFT_SCHEDULES || !shape_ok(g)) return hipErrorInvalidValue;
    const double2* tw;
    hipError_t e = twiddles(&tw);
    if (e != hipSuccess) return e;
    CountSrc cs{src, g.d, {1, 1, 1, 1}, {1, 1, 1, 1}, slots ? 1 : 0, counts, reach};
    for (int k = 0; k < g.d; ++k) {
        cs.M[k] = g.M[k];
        cs.P[k] = g.P[k];
    }
    if (slots && !counts) return hipErrorInvalidValue;
    // the R2C covers the rows inside the counts' box only (prod of the leading M)
    int64_t rows_live = 1;
    for (int k = 0; k + 1 < g.d; ++k) rows_live *= g.M[k];
    e = r2c_last(nullptr, spec, rows_live, g.P[g.d - 1], tw, s, cs, fs);
    if (e != hipSuccess) return e;
    // forward passes over the counts' spectrum, pruned: before the pass along
    // axis a only columns with i_k < M_k (k < a) are nonzero, and only their
    // first M_a entries
    for (int ax = g.d - 2; ax >= 1 && e == hipSuccess; --ax) {
        int64_t outer, inner;
        axis_shape(g, ax, &outer, &inner);
        Prune pr{ax, {1, 1, 1}, {1, 1, 1}, g.M[ax], 0, 0};
        for (int k = 0; k < ax; ++k) {
            pr.P[k] = g.P[k];
            pr.M[k] = g.M[k];
        }
        e = c2c(spec, nullptr, outer, g.P[ax], inner, -1, 0, tw, s, fs, pr);
    }
    if (e != hipSuccess || g.d == 1) return e;
    int64_t outer, inner;
    axis_shape(g, 0, &outer, &inner);
    return c2c(spec, wmix, outer, g.P[0], inner, -1, wmix ? 1 : 0, tw, s, fs,
               Prune{0, {1, 1, 1}, {1, 1, 1}, g.M[0], 0, g.d > 2 ? g.P[0] / 2 + 1 : 0});
}

hipError_t fft_counts_nd(const int64_t* src, int slots, int64_t* counts, double2* spec, const kdefft_grid& g,
                         hipStream_t s) {
    return counts_forward(src, slots, counts, spec, nullptr, g, s, FS_AUTO, nullptr);
}

hipError_t fft_prepare_nd(const int64_t* src, int slots, int64_t* counts, double2* spec, double2* wmix,
                          const kdefft_grid& g, hipStream_t s, int fs, int32_t* reach) {
    hipError_t e = counts_forward(src, slots, counts, spec, wmix, g, s, fs, reach);
    if (e != hipSuccess) return e;
    if (g.d == 1) {
        const int64_t cnt = g.P[0] / 2 + 1;
        hipLaunchKernelGGL(k_abs2, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, spec, wmix, cnt);
        return hipGetLastError();
    }
    const double2* tw;
    e = twiddles(&tw);
    for (int ax = 1; ax + 1 < g.d && e == hipSuccess; ++ax) {
        int64_t outer, inner;
        axis_shape(g, ax, &outer, &inner);
        // l_0 in [0, P_0/2]; the last of these passes fills in the rest
        const int h0 = g.P[0] / 2 + 1;
        Prune pr{0, {1, 1, 1}, {1, 1, 1}, 0, 0, 0};
        const bool last = ax + 2 == g.d;
        if (last) {
            pr.na = ax;
            for (int k = 0; k < ax; ++k) {
                pr.P[k] = g.P[k];
                pr.M[k] = k == 0 ? h0 : g.P[k];
            }
        }
        e = c2c(wmix, nullptr, outer / g.P[0] * h0, g.P[ax], inner, -1, last ? 2 : 0, tw, s, fs, pr);
    }
    return e;
}

hipError_t fft_autocorr_nd(const double2* wmix, double* alag, const kdefft_grid& g, hipStream_t s, int fs) {
    if (!shape_ok(g)) return hipErrorInvalidValue;
    if (fs < 0 || fs >= FFT_SCHEDULES) return hipErrorInvalidValue;
    const double2* tw;
    hipError_t e = twiddles(&tw);
    if (e != hipSuccess) return e;
    // inverting |C|^2 along the leading axes = the forward transform (wmix)
    // read at negated leading indices; then the last-axis inverse.  The result
    // is even, so the rows l_0 in [0, P_0/2] give it all.  Lags with |l| >= M
    // along any axis are zero in exact arithmetic (the counts occupy [0, M))
    // and are stored as exact zeros.
    RowFlip fl{g.d > 1 ? 1 : 0, g.d - 1, {1, 1, 1}, g.M[g.d - 1], {1, 1, 1}};
    for (int k = 0; k + 1 < g.d; ++k) {
        fl.P[k] = g.P[k];
        fl.M[k] = g.M[k];
    }
    const int64_t rows = g.d > 1 ? lead_count(g) / g.P[0] * (g.P[0] / 2 + 1) : 1;
    return c2r_last(wmix, alag, rows, g.P[g.d - 1], tw, s, fl, fs);
}

}  // namespace kdefft
