// One update of the batched minimiser's per-candidate state machine: reads the
// criterion's value and gradient at the trial point, accepts or shortens the
// step and writes the next trial point.
//
// One thread per candidate.  The update is a serial chain, bound by latency:
// the state is read into registers at once (one round trip instead of a load
// per use) and the extents are compile-time, so that nothing is indexed
// through scratch memory.  d = 2, 4 candidates, us an update: 10.0 by itself
// with a runtime q; 3.9 now together with the criterion's assembly.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace kdefft {

// double state per candidate: x[q], g[q], p[q], Hinv[q*q], f, alpha
__host__ __device__ constexpr int min_sw(int q) { return 3 * q + q * q + 2; }

// int32 state per candidate: phase, backtracks of the current line search,
// accepted steps, outcome, accepted steps in a row without a decrease above
// rounding
constexpr int MIN_IS = 8;
enum : int { PH_START = 0, PH_LINE = 1 };

// Armijo constant, backtracking limit, first-step cap
constexpr double C_ARMIJO = 1e-4;
constexpr int MAX_BACK = 60;
constexpr double STEP_CAP = 0.25;   // a new direction moves no entry of x by more than this x max|x|

template <int Q>
__device__ __forceinline__ double min_dot(const double* a, const double* b) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) s = fma(a[i], b[i], s);
    return s;
}

template <int Q>
__device__ __forceinline__ double min_amax(const double* a) {
    double m = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) m = fmax(m, fabs(a[i]));
    return m;
}

// State of candidate b in registers.
template <int Q>
struct MinState {
    double x[Q], g[Q], p[Q], Hi[Q * Q], xt[Q], f, alpha;
    int phase, back, acc, outcome, flat;
    bool bad;   // the criterion rejected the trial point
    __device__ __forceinline__ MinState(const MinStep& a, int64_t b) {
        const double* st = a.st + b * min_sw(Q);
        const int32_t* is = a.ist + MIN_IS * b;
        phase = is[0];
        back = is[1];
        acc = is[2];
        outcome = is[3];
        flat = is[4];
        bad = a.stt && a.stt[b] != 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            x[i] = st[i];
            g[i] = st[Q + i];
            p[i] = st[2 * Q + i];
            xt[i] = a.xt[b * Q + i];
        }
#pragma unroll
        for (int i = 0; i < Q * Q; ++i) Hi[i] = st[3 * Q + i];
        f = st[3 * Q + Q * Q];
        alpha = st[3 * Q + Q * Q + 1];
    }
};

// Candidate b: value fb and gradient gb at its trial point.
template <int Q>
__device__ __forceinline__ void min_step(const MinStep& a, int64_t b, const MinState<Q>& now, double fb,
                                         const double* gb) {
    double* st = a.st + b * min_sw(Q);
    int32_t* is = a.ist + MIN_IS * b;
    double* xt_out = a.xt + b * Q;
    const auto &x = now.x, &g = now.g, &xt = now.xt;
    const double f = now.f;
    const int back = now.back, acc = now.acc, flat = now.flat;
    double p[Q], Hi[Q * Q], alpha = now.alpha;
#pragma unroll
    for (int i = 0; i < Q; ++i) p[i] = now.p[i];
#pragma unroll
    for (int i = 0; i < Q * Q; ++i) Hi[i] = now.Hi[i];
    const auto trial_at_x = [&](const double* at) {
#pragma unroll
        for (int i = 0; i < Q; ++i) xt_out[i] = at[i];
    };
    if (now.outcome != KDEFFT_MIN_RUNNING) {
        trial_at_x(x);
        return;
    }
    bool ok = !now.bad && isfinite(fb);
#pragma unroll
    for (int i = 0; i < Q; ++i) ok = ok && isfinite(gb[i]);
    const double gp = min_dot<Q>(g, p);
    const bool start = now.phase == PH_START;
    if (!start && !(ok && fb <= f + C_ARMIJO * alpha * gp)) {
        // rejected: shorten the step to the minimiser of the quadratic through
        // f, the slope gp and the trial value, kept within [0.1, 0.5] of the step
        is[1] = back + 1;
        if (back + 1 > MAX_BACK) {
            is[3] = KDEFFT_MIN_STALLED;
            trial_at_x(x);
            return;
        }
        double an = 0.25 * alpha;
        if (ok) {
            const double den = 2.0 * (fb - f - alpha * gp);
            an = den > 0.0 ? -gp * alpha * alpha / den : 0.5 * alpha;
            an = fmin(fmax(an, 0.1 * alpha), 0.5 * alpha);
        }
        st[3 * Q + Q * Q + 1] = an;
#pragma unroll
        for (int i = 0; i < Q; ++i) xt_out[i] = x[i] + an * p[i];
        return;
    }
    // the start, or an accepted step: the trial point becomes the point
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        st[i] = xt[i];
        st[Q + i] = gb[i];
    }
    st[3 * Q + Q * Q] = fb;
    if (start) {
        if (!ok) {
            is[3] = KDEFFT_MIN_BAD_START;
            return;
        }
#pragma unroll
        for (int i = 0; i < Q * Q; ++i) Hi[i] = (i % (Q + 1)) == 0 ? 1.0 : 0.0;
    } else {
        // BFGS update of the inverse Hessian with s = xt - x, y = gt - g
        double sv[Q], yv[Q], hy[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            sv[i] = xt[i] - x[i];
            yv[i] = gb[i] - g[i];
        }
        const double sy = min_dot<Q>(sv, yv), yy = min_dot<Q>(yv, yv);
        // the update needs curvature well above the rounding of s and y
        if (yy > 0.0 && sy > 1e-10 * sqrt(min_dot<Q>(sv, sv) * yy)) {
            if (acc == 0) {
                // first accepted step: the identity scaled to the observed curvature
                const double sc = sy / yy;
#pragma unroll
                for (int i = 0; i < Q * Q; ++i) Hi[i] *= sc;
            }
#pragma unroll
            for (int i = 0; i < Q; ++i) hy[i] = min_dot<Q>(Hi + i * Q, yv);
            const double rho = 1.0 / sy;
            const double c = rho * (1.0 + rho * min_dot<Q>(yv, hy));
#pragma unroll
            for (int i = 0; i < Q; ++i)
#pragma unroll
                for (int j = 0; j < Q; ++j)
                    Hi[i * Q + j] += c * sv[i] * sv[j] - rho * (hy[i] * sv[j] + sv[i] * hy[j]);
        }
        // a decrease within a few roundings of f is no decrease: two such
        // accepted steps in a row end the search (float64 offers no more)
        const int flat1 = f - fb <= 8.8817841970012523e-16 * fabs(f) ? flat + 1 : 0;
        is[4] = flat1;
        is[2] = acc + 1;
        // first-order test, invariant to the scales of f and of x
        const bool conv = min_amax<Q>(gb) * min_amax<Q>(xt) <= a.tol * fabs(fb);
        if (conv || flat1 >= 2) {
            is[3] = conv ? KDEFFT_MIN_CONVERGED : KDEFFT_MIN_STALLED;
            trial_at_x(xt);
            return;
        }
    }
    // the next direction p = -Hinv g (a steepest-descent restart if that is not
    // a descent direction), first step length 1 capped so that no entry moves
    // by more than STEP_CAP x max|x|
#pragma unroll
    for (int i = 0; i < Q; ++i) p[i] = -min_dot<Q>(Hi + i * Q, gb);
    if (!(min_dot<Q>(gb, p) < 0.0)) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
#pragma unroll
            for (int j = 0; j < Q; ++j) Hi[i * Q + j] = i == j ? 1.0 : 0.0;
            p[i] = -gb[i];
        }
    }
    const double pn = min_amax<Q>(p), xn = min_amax<Q>(xt);
    alpha = pn > STEP_CAP * xn && pn > 0.0 ? STEP_CAP * xn / pn : 1.0;
    st[3 * Q + Q * Q + 1] = alpha;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        st[2 * Q + i] = p[i];
        xt_out[i] = xt[i] + alpha * p[i];
    }
#pragma unroll
    for (int i = 0; i < Q * Q; ++i) st[3 * Q + i] = Hi[i];
    is[0] = PH_LINE;
    is[1] = 0;
}

}  // namespace kdefft
