"""Batched criteria on thin grids, where the items of a launch over B candidates
and over B plus the datasets' constant terms differ most, in a workspace of
exactly the size asked for: the bytes behind it stay as they were, and the
results are those of calls on a few candidates each.

Tolerance: the split into items differs, so the order of summation does:
rounding of a few hundred summed terms."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth

from _gpu_util import log, mixture_sample, spd

pytestmark = pytest.mark.gpu

GUARD = 1 << 18


def _vech(B, d, seed):
    rng = np.random.default_rng(seed)
    H = synth.random_H_haar(B, d, rng)
    return torch.from_numpy(synth.vech_chol(H)).cuda()


@pytest.mark.parametrize("M,B,nds", [([4, 155], 522, 1), ([6, 511], 266, 1), ([2, 372], 569, 1),
                                     ([17, 2, 121], 6, 54)], ids=str)
def test_workspace_end(kf, gpu, M, B, nds):
    d = len(M)
    q = d * (d + 1) // 2
    dss = [kf.Dataset(torch.from_numpy(mixture_sample(300 + j, d, 700 + j)).to(gpu), spd(d, 710, 0.05), M=M)
           for j in range(nds)]
    v = _vech(B, d, 720)
    lib = kf._lib.load()
    per = [B // nds + (1 if j < B % nds else 0) for j in range(nds)]
    off = (C.c_int64 * (nds + 1))(*np.concatenate([[0], np.cumsum(per)]).tolist())
    arr = (kf._lib.Dataset * nds)(*[ds.desc for ds in dss])
    need = C.c_size_t()
    kf._lib.check(lib.kdefft_ws_bytes(C.byref(dss[0].shape_grid), kf._lib.OP_SCV_BATCH, 2, B, C.byref(need)), "bytes")
    buf = torch.full((need.value + 256 + GUARD,), 0xA5, dtype=torch.uint8, device=gpu)
    at = (-buf.data_ptr()) % 256
    stream = torch.cuda.current_stream().cuda_stream
    w = torch.linspace(0.5, 2.0, B, dtype=torch.float64, device=gpu)
    obj, grad, adj = (torch.empty(s, dtype=torch.float64, device=gpu) for s in ((B,), (B, q), (B, q)))
    lobj, lgrad = torch.empty_like(obj), torch.empty_like(grad)
    args = (arr, nds, off, v.data_ptr())
    end = (buf.data_ptr() + at, need.value, stream)
    log(f"[extent] M={M} B={B} datasets {nds}")
    kf._lib.check(lib.kdefft_scv_batch(*args, obj.data_ptr(), grad.data_ptr(), None, *end), "scv")
    kf._lib.check(lib.kdefft_scv_adjoint(*args, w.data_ptr(), adj.data_ptr(), *end), "adjoint")
    kf._lib.check(lib.kdefft_crit_batch(*args, kf.CRIT_LSCV, 0, lobj.data_ptr(), lgrad.data_ptr(), None, *end), "lscv")
    assert bool((buf[:at] == 0xA5).all()) and bool((buf[at + need.value:] == 0xA5).all())
    start = 0
    for j, ds in enumerate(dss):
        for s in range(start, start + per[j], 40):
            e = min(s + 40, start + per[j])
            for got_o, got_g, (o, g) in ((obj, grad, kf.scv([ds], v[s:e])), (lobj, lgrad, kf.crit([ds], v[s:e], "lscv"))):
                assert torch.allclose(got_o[s:e], o, rtol=1e-11, atol=0)
                assert torch.allclose(got_g[s:e], g, rtol=1e-10, atol=1e-13 * float(g.abs().max()))
        start += per[j]
    assert torch.allclose(adj, grad * w[:, None], rtol=1e-10, atol=1e-13 * float(grad.abs().max()))


def test_tuner_workspace_end(kf, gpu):
    """The tuner's launches (256 candidates, with and without the constant
    term) at the benchmark's shape stay inside the workspace asked for."""
    d, M = 2, [256, 256]
    ds = kf.Dataset(torch.from_numpy(mixture_sample(20000, d, 730)).to(gpu), spd(d, 731, 0.02), M=M)
    lib = kf._lib.load()
    need = C.c_size_t()
    kf._lib.check(lib.kdefft_ws_bytes(C.byref(ds.shape_grid), kf._lib.OP_AUTOTUNE, 2, 256, C.byref(need)), "bytes")
    buf = torch.full((need.value + 256 + GUARD,), 0xA5, dtype=torch.uint8, device=gpu)
    at = (-buf.data_ptr()) % 256
    P = list(ds.shape_grid.P[:d])
    keys = [(k, 2) for k in (kf.FUN_SCV_OBJ, kf.FUN_SCV_OBJGRAD, kf.FUN_SCV_GRAD)] + [(kf.FUN_PSI, 4)]
    saved = [(k, r, kf.get_row_launch(k, d, r, P[-1])) for k, r in keys]
    saved_fft = kf.get_fft_schedule(P)
    try:
        kf._lib.check(lib.kdefft_autotune(C.byref(ds.desc), buf.data_ptr() + at, need.value, None,
                                          torch.cuda.current_stream().cuda_stream), "autotune")
        log("[extent] tuner " + lib.kdefft_last_error_detail().decode().replace("\n", "; "))
    finally:
        for k, r, (variant, blocks) in saved:
            kf.set_row_launch(k, d, r, P[-1], variant, blocks)
        kf.set_fft_schedule(P, saved_fft)
    assert bool((buf[:at] == 0xA5).all()) and bool((buf[at + need.value:] == 0xA5).all())
