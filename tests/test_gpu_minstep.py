"""The minimiser's update in every dimension, inside the criterion's assembly
(SCV) and by itself (PI), against the same update written in numpy on the
criterion's own values and gradients.

Tolerance: the two differ by the rounding of the update (1e-16, contracted or
not) and of the launches' values; a BFGS direction amplifies a relative error by
the condition of the inverse Hessian, which over eight evaluations from these
starts stays below 1e6 in steps of at most a quarter of x, so 1e-8 of max|x|."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EVALS = 8


TOL = 1e-9


def _reference(fun, x0, done):
    """One candidate: fun(x) -> (f, g); done: the outcomes (running, converged,
    stalled).  Returns x, f, outcome, accepted steps."""
    q = len(x0)
    xt, x, f, g, p, H, alpha, acc, flat = x0.copy(), None, None, None, None, None, None, 0, 0

    def direction():
        nonlocal H, p, alpha, xt
        p = -H @ g
        if not g @ p < 0:
            H, p = np.eye(q), -g
        pn, xn = np.abs(p).max(), np.abs(x).max()
        alpha = 0.25 * xn / pn if pn > 0.25 * xn else 1.0
        xt = x + alpha * p

    for _ in range(EVALS):
        ft, gt = fun(xt)
        if x is None:
            x, f, g, H = xt, ft, gt, np.eye(q)
            direction()
            continue
        gp = g @ p
        if ft <= f + 1e-4 * alpha * gp:
            s, y = xt - x, gt - g
            sy, yy = s @ y, y @ y
            if yy > 0 and sy > 1e-10 * np.sqrt(s @ s * yy):
                if acc == 0:
                    H = H * (sy / yy)
                hy = H @ y
                rho = 1 / sy
                H = H + rho * (1 + rho * (y @ hy)) * np.outer(s, s) - rho * (np.outer(hy, s) + np.outer(s, hy))
            flat = flat + 1 if f - ft <= 4 * np.finfo(float).eps * abs(f) else 0
            x, f, g = xt, ft, gt
            acc += 1
            if np.abs(g).max() * np.abs(x).max() <= TOL * abs(f):
                return x, f, done[1], acc
            if flat >= 2:
                return x, f, done[2], acc
            direction()
            continue
        den = 2 * (ft - f - alpha * gp)
        an = -gp * alpha * alpha / den if den > 0 else 0.5 * alpha
        alpha = min(max(an, 0.1 * alpha), 0.5 * alpha)
        xt = x + alpha * p
    return x, f, done[0], acc


@pytest.mark.parametrize("crit", ["scv", "pi"])
@pytest.mark.parametrize("d", [1, 2, 3, 4])
def test_update(d, crit):
    import paper_1511_07482_amd as kf
    rng = np.random.default_rng(70 + d)
    n, M, B = 3000, {1: 128, 2: 48, 3: 24, 4: 12}[d], 5
    X = torch.tensor(rng.standard_normal((n, d)) * (1 + 0.3 * np.arange(d)), device="cuda")
    ds = kf.Dataset(X, 0.15 * np.eye(d), M=[M] * d)
    starts = []
    for _ in range(B):
        L = np.tril(0.08 * rng.standard_normal((d, d)))
        np.fill_diagonal(L, rng.uniform(0.3, 0.9, d))
        starts.append(np.concatenate([L[j:, j] for j in range(d)]))
    v0 = torch.tensor(np.array(starts), device="cuda")
    print(f"[minstep] d={d} {crit}", flush=True)
    if crit == "scv":
        def call(v):
            return kf.scv([ds], v)[:2]
        x, f, info = kf.minimize(v0, "scv", datasets=[ds], evals=EVALS, tol=TOL)
    else:
        psi4 = kf.psi_batch([ds], [0.3 * np.eye(d)], 4)

        def call(v):
            return kf.pi(psi4, [n], v)[:2]
        x, f, info = kf.minimize(v0, "pi", psi4=psi4, ns=[n], evals=EVALS, tol=TOL)

    def fun(xx):
        o, g = call(torch.tensor(xx[None], device="cuda"))
        return float(o[0]), g[0].cpu().numpy()

    moved = 0
    for b in range(B):
        xr, fr, outcome, acc = _reference(fun, starts[b], (kf.MIN_RUNNING, kf.MIN_CONVERGED, kf.MIN_STALLED))
        assert (int(info[b, 0]), int(info[b, 1])) == (outcome, acc)
        assert np.abs(x[b].cpu().numpy() - xr).max() <= 1e-8 * np.abs(xr).max()
        assert abs(float(f[b]) - fr) <= 1e-8 * abs(fr)
        moved += acc
    assert moved > 0
