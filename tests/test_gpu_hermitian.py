"""The count transform computes half of the mixed spectrum and of the lag array
and fills in the rest by symmetry: both in full against float64 FFTs on the CPU,
for every number of axes, unequal extents and each schedule.

Tolerance: a transform of N values loses at most about log2(N) roundings of the
largest partial result: 16 log2(prod P) 2^-53 of the largest entry."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [(1, [9]), (2, [3, 40]), (2, [33, 17]), (2, [130, 260]), (3, [9, 20, 33]), (3, [33, 60, 40]),
         (3, [64, 64, 64]), (4, [5, 9, 17, 8]), (4, [17, 12, 20, 30])]


@pytest.mark.parametrize("d,M", CASES)
def test_symmetric_half(d, M):
    import paper_1511_07482_amd as kf
    rng = np.random.default_rng(sum(M))
    X = torch.tensor(rng.standard_normal((2000, d)), device="cuda")
    ds = kf.Dataset(X, 0.05 * np.eye(d), M=M)
    P = list(ds.shape_grid.P[:d])
    print(f"[hermitian] d={d} M={M} P={P}", flush=True)
    c = ds.counts().cpu().numpy().astype(np.float64) * 2.0 ** -40
    pad = np.zeros(P)
    pad[tuple(slice(0, m) for m in M)] = c
    C = np.fft.rfftn(pad)
    W = np.abs(C) ** 2 + 0j
    for k in range(d - 1):
        W = np.fft.fft(W, axis=k)
    lag = np.fft.irfftn(np.abs(C) ** 2, s=P, axes=range(d)) * np.prod(P)
    tol = 16 * np.log2(np.prod(P)) * 2.0 ** -53
    shape = tuple(P[:-1]) + (P[-1] // 2 + 1,)
    start = ds.desc.wmix - ds.mem.data_ptr()

    def check():
        w = ds.mem[start:start + 16 * int(np.prod(shape))].view(torch.complex128).view(shape).cpu().numpy()
        assert np.abs(w - W).max() <= tol * np.abs(W).max()
        a = ds.lag_array().cpu().numpy()
        assert np.abs(a - lag).max() <= tol * np.abs(lag).max()
        for k in range(d):   # exact zeros beyond the counts
            dead = np.arange(P[k])[M[k]:P[k] - M[k] + 1]
            assert not np.take(a, dead, axis=k).any()

    check()
    try:
        for fs in range(6):
            kf.set_fft_schedule(P, fs)
            ds.transform()
            check()
    finally:
        kf.set_fft_schedule(P, -1)
