"""Bandwidths far below a grid step in some or all directions (down to 1e-40 of
it): only the lags at distance zero along those axes count, and the others'
weights are exactly zero, however far the exponent.  Against the oracle's
binned criteria, per entry under the near-zero rule; the bar of the other
criterion tests, 1e-11."""
import numpy as np
import pytest
import torch

import synth
from oracle import eta, grid, linbin

from _gpu_util import check_z16, log, mixture_sample, oracle_autocorr, spd

pytestmark = pytest.mark.gpu

STDS = [[1e-36], [1e-40], [1e-38, 1e-40], [1e-40, 0.4], [0.4, 1e-40], [1e-40, 1e-38, 1e-41], [0.5, 0.4, 1e-40],
        [1e-40, 0.3, 0.5], [0.4, 1e-40, 0.5]]


@pytest.mark.parametrize("stds", STDS, ids=lambda s: "x".join(map(str, s)))
def test_narrow_bandwidths(kf, gpu, stds):
    d, n = len(stds), 300
    for M in ([9, 12, 10][:d], [20, 18, 19][:d]):   # the walked axis padded to at least 16, and to less (d = 1: none)
        X = mixture_sample(n, d, 750 + d)
        G = spd(d, 751, 0.05)
        g = grid.plan_auto(X, G, M)
        counts, _ = linbin.linbin(X, g)
        A = oracle_autocorr(linbin.counts_to_real(counts))
        H = np.diag(np.square(stds))
        ds = kf.Dataset(torch.from_numpy(X).to(gpu), G, M=M)
        v = torch.from_numpy(synth.vech_chol(H[None])).to(gpu)
        log(f"[narrow] M={M} {stds}")
        for exact in (False, True):
            obj, grad = kf.crit([ds], v, "lscv_exact" if exact else "lscv")
            want, wgrad = eta.lscv_binned(A, n, g, H, exact)
            scale, sgrad = eta.lscv_binned_scales(A, n, g, H, exact)
            got = grad[0].cpu().numpy()
            check_z16([float(obj[0])], [want], [scale], what=f"{stds} objective")
            none = sgrad == 0   # a sum without terms
            assert np.all(got[none] == 0) and np.all(wgrad[none] == 0), f"{stds} gradient {got}"
            check_z16(got[~none], wgrad[~none], sgrad[~none], what=f"{stds} gradient")
        for r in (0, 1):
            q = float(kf.crit([ds], v, "qr", r, grad=False)[0])
            check_z16([q], [eta.qr_binned(A, n, g, H, r)],
                      [eta.vstat_binned(A, n, g, [(1.0, H)], r, absval=True)], what=f"Q_{r} {stds}")
