"""Data without a finite range leave a dataset without a grid (every point out
of it): psi_r, Q_r and LSCV_r for r >= 1 of it are NaN, not the sum of no lags."""
import numpy as np
import pytest
import torch

import synth

from _gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4])
def test_no_grid_gives_nan(kf, gpu, d):
    for axis in range(d):
        X = np.random.default_rng(11).normal(size=(200, d))
        X[5, axis] = np.inf
        ds = kf.Dataset(torch.from_numpy(X).to(gpu), 0.1 * np.eye(d), M=6)
        assert ds.out_of_grid() == 200
        log(f"[nonfinite] d={d} axis {axis}")
        for r in (0, 2, 4):
            assert bool(torch.isnan(kf.psi_batch([ds], [0.1 * np.eye(d)], r)).all()), r
        v = torch.from_numpy(synth.vech_chol(np.stack([0.1 * np.eye(d), 0.3 * np.eye(d)]))).to(gpu)
        for crit, rs in (("qr", (0, 1, 2)), ("lscv", (1, 2)), ("lscv_exact", (1, 2))):
            for r in rs:
                assert bool(torch.isnan(kf.crit([ds], v, crit, r, grad=False)).all()), (crit, r)
