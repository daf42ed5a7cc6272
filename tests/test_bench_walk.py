"""The benchmark's count of the lags the column walk covers (CPU): at least the
lags of the half set inside the cut, at most those rounded out to whole runs."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("M,scale", [([64, 40], 1.0), ([33, 64], 0.02), ([200, 31], 40.0), ([12, 40, 17], 1.0),
                                     ([6, 9, 24, 7], 3.0)])
def test_lags_of_the_column_walk(M, scale):
    d = len(M)
    rng = np.random.default_rng(sum(M))
    A = rng.standard_normal((d, d))
    G = 0.05 * (A @ A.T / d + 0.5 * np.eye(d))
    L = np.linalg.cholesky(scale * (A.T @ A / d + 0.3 * np.eye(d)))
    delta = [8.0 / (m - 1) for m in M]
    reach = bench.data_reach([0.4] * d, [6.0] * d, M, delta)
    assert all(r <= m - 1 for r, m in zip(reach, M)) and min(reach) >= 1
    for cand in (L, None):
        S = 2 * G if cand is None else 2 * L @ L.T + 2 * G
        P = np.linalg.inv(S)
        lags = [np.arange(0 if k == 0 else -reach[k], reach[k] + 1) for k in range(d)]
        x = [v * h for v, h in zip(np.meshgrid(*lags, indexing="ij"), delta)]
        live = sum(P[i, j] * x[i] * x[j] for i in range(d) for j in range(d)) <= 2 * np.log(1e30)
        count = bench.column_walk_lags(M, delta, reach, G, cand)
        columns = int(live.any(axis=d - 2).sum())
        # whole runs of 8, and a run more where an end is rounded to the next lag
        # (a column whose interval holds no lag at all may be met too)
        near = np.prod([2 * r + 3 for k, r in enumerate(reach) if k != d - 2])
        assert live.sum() <= count <= live.sum() + 16 * columns + 8 * near
