"""The column walk (SCV families: launch variants 5 and 6; psi_r; eta_r of low
order) at the edges of its units -- 16-lag blocks of the last axis, runs of 8 rows, segments of 64
rows, walked axes shorter than a run -- against the oracle's
binned criterion on the same counts, for narrow kernels (a fraction of a grid
step: evaluated lag by lag), ordinary and wide ones.

Tolerance: the parity bar of the other SCV tests, 1e-11 relative per entry
under the near-zero rule (rounding of a few thousand summed terms is below
1e-13 of their absolute sum)."""
import numpy as np
import pytest
import torch

import synth
from oracle import binned, eta, grid, linbin, multiindex

from _gpu_util import assert_psi_close, check_scv, check_z16, log, mixture_sample, oracle_autocorr, spd

pytestmark = pytest.mark.gpu

# nodes per axis; the walked axis is the second last, the lanes the last
SHAPES = [
    [2], [300],
    [2, 2], [4, 16], [5, 9], [8, 17], [9, 33], [33, 5], [65, 16], [40, 7],
    [3, 2, 3], [9, 4, 17], [2, 33, 8], [5, 34, 9],
    [2, 2, 3, 2], [3, 4, 5, 16], [9, 3, 33, 4],
]


@pytest.mark.parametrize("M", SHAPES, ids=lambda m: "x".join(map(str, m)))
def test_column_walk_edges(kf, gpu, M):
    d = len(M)
    n = 400
    X = mixture_sample(n, d, 500 + d)
    G = spd(d, 510 + d, 0.05)
    g = grid.plan_auto(X, G, M)
    counts, skipped = linbin.linbin(X, g)
    assert skipped == 0
    A = oracle_autocorr(linbin.counts_to_real(counts))
    rng = np.random.default_rng(520 + d)
    base = synth.random_H_haar(1, d, rng)[0] if d > 1 else np.array([[0.4]])
    H = np.stack([base * s for s in (1e-4, 0.02, 0.3, 1.0, 30.0)])
    ds = kf.Dataset(torch.from_numpy(X).to(gpu), G, M=M)
    v = torch.from_numpy(synth.vech_chol(H)).to(gpu)
    N = ds.shape_grid.P[d - 1]
    w = torch.linspace(0.5, 2.0, len(H), dtype=torch.float64, device=gpu)
    for variant, blocks in ((5, -1), (6, 0), (5, 3)):
        log(f"[cols] M={M} variant {variant} grid {blocks}")
        with kf.row_launch([1, 2, 3], d, 2, N, variant, blocks):
            obj, grad = kf.scv([ds], v)
            only = kf.scv([ds], v, grad=False)
            adj = kf.scv_adjoint([ds], v, w)
        for b in range(len(H)):
            check_scv(float(obj[b]), grad[b].cpu().numpy(), A, n, g, H[b], G, what=f"M={M} b={b}")
            check_scv(float(only[b]), (adj[b] / w[b]).cpu().numpy(), A, n, g, H[b], G, what=f"M={M} b={b} adjoint")


@pytest.mark.parametrize("M", SHAPES, ids=lambda m: "x".join(map(str, m)))
def test_derivative_families_edges(kf, gpu, M):
    """psi_r up to the largest order, Q_r and LSCV_r of the orders the walk serves."""
    d = len(M)
    n = 300
    X = mixture_sample(n, d, 570 + d)
    G = spd(d, 571 + d, 0.05)
    g = grid.plan_auto(X, G, M)
    counts, _ = linbin.linbin(X, g)
    A = oracle_autocorr(linbin.counts_to_real(counts))
    ds = kf.Dataset(torch.from_numpy(X).to(gpu), G, M=M)
    S = [G * s for s in (1e-3, 1.0, 40.0)]
    for r in (0, 2, {1: 8, 2: 8, 3: 6, 4: 4}[d]):
        for k, got in enumerate(kf.psi_batch([ds] * 3, S, r).cpu().numpy()):
            log(f"[cols] psi M={M} r={r} {k}")
            sabs = binned.abs_scale(A, n, g, S[k], multiindex.unique_alphas(d, r))
            assert_psi_close(got, binned.psi(A, n, g, S[k], r), sabs, what=f"M={M} r={r} {k}")
    v = torch.from_numpy(synth.vech_chol(np.stack(S))).to(gpu)
    for r in (0, 1, 2):
        q = kf.crit([ds], v, "qr", r, grad=False).cpu().numpy()
        for k in range(3):
            log(f"[cols] Q_{r} M={M} {k}")
            check_z16([q[k]], [eta.qr_binned(A, n, g, S[k], r)],
                      [eta.vstat_binned(A, n, g, [(1.0, S[k])], r, absval=True)], what=f"Q_{r} {k}")
        for exact in (False, True):
            if r == 0:
                continue
            c = kf.crit([ds], v, "lscv_exact" if exact else "lscv", r, grad=False).cpu().numpy()
            for k in range(3):
                check_z16([c[k]], [eta.lscv_r_binned(A, n, g, S[k], r, exact)],
                          [eta.lscv_abs_scale(A, n, g, S[k], r, exact)], what=f"LSCV_{r} {exact} {k}")


def test_column_walk_item_order(kf, gpu):
    """Several datasets and more candidates than resident blocks (items dealt
    part by part over the dies), against one call per candidate group."""
    d, M = 3, [17, 12, 20]
    dss = [kf.Dataset(torch.from_numpy(mixture_sample(500 + 100 * j, d, 530 + j)).to(gpu), spd(d, 540 + j, 0.05), M=M)
           for j in range(3)]
    H = synth.random_H_haar(150, d, np.random.default_rng(550))
    v = torch.from_numpy(synth.vech_chol(H)).to(gpu)
    per = [20, 0, 130]
    obj, grad = kf.scv(dss, v, per_ds=per)
    at = 0
    for ds, b in zip(dss, per):
        for s in range(at, at + b, 7):
            e = min(s + 7, at + b)
            o, g = kf.scv([ds], v[s:e])
            # the split into items differs, so the summation order does: rounding of the sums only
            assert torch.allclose(o, obj[s:e], rtol=1e-11, atol=0)
            assert torch.allclose(g, grad[s:e], rtol=1e-10, atol=1e-13 * float(g.abs().max()))
        at += b


def test_transform_of_replaced_counts(kf, gpu):
    """The walk is cut to the lags the binned data reach; after the counts are
    replaced (to the grid's corners) and transformed again it covers them all."""
    d, M, n = 2, [24, 30], 400
    X = mixture_sample(n, d, 560)
    G = spd(d, 561, 0.3)
    ds = kf.Dataset(torch.from_numpy(X).to(gpu), G, M=M)
    g = ds.grid
    c = torch.zeros(M, dtype=torch.int64)
    c[0, 0] = c[-1, -1] = c[0, -1] = c[-1, 0] = n // 4 << 40
    at = ds.desc.counts - ds.mem.data_ptr()
    ds.mem[at:at + 8 * c.numel()] = c.view(-1).view(torch.uint8).to(gpu)
    ds.transform()
    H = np.stack([np.eye(2) * s for s in (0.5, 40.0, 900.0)])
    obj, grad = kf.scv([ds], torch.from_numpy(synth.vech_chol(H)).to(gpu))
    A = oracle_autocorr(linbin.counts_to_real(c.numpy()))
    go = grid.plan_auto(X, G, M)
    assert list(g.M[:d]) == M
    for b in range(len(H)):
        check_scv(float(obj[b]), grad[b].cpu().numpy(), A, n, go, H[b], G, what=f"replaced counts b={b}")
