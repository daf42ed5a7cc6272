"""The plain path's convolution passes (kernel grids taken together, the slices
at negative axis-0 lags as conjugates, the inverse stored inside the counts'
box): psi_r against the oracle at the edges of their tiles and rows, and a call
whose kernel grids need several batches against the fused path.

Tolerance: the parity bar of the other psi tests, 1e-11 relative per entry
under the near-zero rule."""
import numpy as np
import pytest
import torch

from oracle import binned, grid, linbin, multiindex

from _gpu_util import assert_psi_close, log, mixture_sample, oracle_autocorr, spd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [[2], [130], [2, 2], [3, 130], [130, 3], [70, 66], [2, 5, 3], [5, 2, 40], [3, 2, 4, 2]],
                         ids=lambda m: "x".join(map(str, m)))
def test_psi_plain_edges(kf, gpu, M):
    d, n = len(M), 250
    X = mixture_sample(n, d, 700 + d)
    G = spd(d, 701 + d, 0.1)
    g = grid.plan_auto(X, G, M)
    counts, _ = linbin.linbin(X, g)
    A = oracle_autocorr(linbin.counts_to_real(counts))
    for r in (0, 4):
        log(f"[conv] M={M} r={r}")
        got = kf.psi(torch.from_numpy(X).to(gpu), G, r, M=M).cpu().numpy()
        sabs = binned.abs_scale(A, n, g, G, multiindex.unique_alphas(d, r))
        assert_psi_close(got, binned.psi(A, n, g, G, r), sabs, what=f"M={M} r={r}")


def test_psi_plain_in_batches(kf, gpu):
    """15 grids of 17 MB each: more than one batch (64 MiB)."""
    d, M = 3, [64, 64, 64]
    X = torch.from_numpy(mixture_sample(3000, d, 710)).to(gpu)
    G = spd(d, 711, 0.1)
    a = kf.psi(X, G, 4, M=M).cpu().numpy()
    b = kf.psi(X, G, 4, M=M, mode="fused").cpu().numpy()
    # two routes for the same sums, rounding apart
    assert np.abs(a - b).max() <= 1e-11 * np.abs(b).max()
