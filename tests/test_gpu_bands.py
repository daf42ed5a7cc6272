"""Binning by bands of nodes in LDS against the host oracle and against the
scattered form: the counts are integers and must agree exactly, so no tolerance
applies.  Sizes: one band, a band boundary inside a row, the most bands that are
taken, a last part that is short or empty, out-of-grid and tied points, and both
sides of the rule on the number of points."""
import numpy as np
import pytest
import torch

from oracle import linbin

pytestmark = pytest.mark.gpu

CASES = [  # d, M per axis, n
    (1, [64], 10000), (1, [2048], 10001),
    (2, [142, 143], 61000),          # 20306 nodes: one band
    (2, [143, 143], 61400),          # 20449: two bands, cut inside a row
    (2, [300, 61], 70001),
    (2, [404, 404], 489700),         # 163216: eight bands
    (3, [27, 27, 27], 20001), (3, [54, 53, 57], 163200),
    (4, [8, 8, 8, 8], 10000), (4, [20, 20, 20, 20], 40011),
    (2, [143, 143], 61300),          # just below the rule: scattered
]


@pytest.mark.parametrize("d,M,n", CASES)
def test_band_counts_exact(d, M, n):
    import paper_1511_07482_amd as kf
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d))
    X[: n // 50] = X[0]                       # tied points
    lo, hi = X.min(0) - 0.1, X.max(0) + 0.1
    lo[0] += 0.6                              # some points fall outside, axis 0 and the last axis
    hi[-1] -= 0.5
    g = kf.grid_plan(M, lo, hi)
    print(f"[bands] d={d} M={M} n={n}", flush=True)
    Xd = torch.tensor(X, device="cuda")
    want, skipped = linbin.linbin(X, g.to_dict())
    counts, nout = kf.linbin(Xd, g)
    assert int(nout.item()) == skipped > 0
    assert np.array_equal(counts.cpu().numpy().reshape(want.shape), want)


@pytest.mark.parametrize("d,M,n", [(1, [64], 10000), (2, [143, 143], 61400), (3, [27, 27, 27], 20001),
                                   (4, [8, 8, 8, 9], 10000),
                                   # through the corner slots: short, odd and full rows
                                   (1, [65], 500), (2, [130, 3], 700), (2, [3, 256], 9000), (3, [5, 33, 64], 900),
                                   (4, [3, 7, 4, 31], 900), (4, [4, 5, 6, 32], 2000)])
def test_band_preparation(d, M, n):
    """The preparation on the device's own grid, eager and replayed on new data."""
    import paper_1511_07482_amd as kf
    rng = np.random.default_rng(n)
    Xs = [torch.tensor(rng.standard_normal((n, d)) * (1 + j), device="cuda") for j in range(3)]
    G = np.eye(d) * 0.05
    print(f"[bands] prepare d={d} M={M} n={n}", flush=True)
    X = Xs[0].clone()
    kf.Dataset(X, G, M=M)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ds = kf.Dataset(X, G, M=M)
        c, lag = ds.counts(), ds.lag_array()
    for Y in Xs:
        X.copy_(Y)
        graph.replay()
        torch.cuda.synchronize()
        want, skipped = linbin.linbin(Y.cpu().numpy(), kf.grid_auto(Y, G, M).to_dict())
        assert skipped == 0
        assert np.array_equal(c.cpu().numpy().reshape(want.shape), want)
        eager = kf.Dataset(Y, G, M=M)
        assert torch.equal(eager.lag_array(), lag)
