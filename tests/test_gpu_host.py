"""Calls whose candidates and datasets span several launches, on converted and
strided inputs: each part's addresses against one call per dataset, which must
agree exactly (the same kernels on the same values)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_parts_and_inputs():
    import paper_1511_07482_amd as kf
    from paper_1511_07482_amd import _lib
    rng = np.random.default_rng(5)
    nds = _lib.MAX_BATCH_DS + 3
    per = [int(c) for c in rng.integers(0, 4, nds)]
    per[0], per[-1] = 2, 3
    dss = [kf.Dataset(torch.tensor(rng.standard_normal((300, 2)), device="cuda"), 0.2 * np.eye(2), M=[16, 12])
           for _ in range(nds)]
    B = sum(per)
    v = torch.tensor(np.column_stack([rng.uniform(0.3, 0.9, B), 0.1 * rng.standard_normal(B),
                                      rng.uniform(0.3, 0.9, B)]), device="cuda")
    wide = torch.empty(B, 6, dtype=torch.float64, device="cuda")
    wide[:, ::2] = v
    go = torch.tensor(rng.standard_normal(B), device="cuda")
    forms = {"contiguous": v, "strided": wide[:, ::2], "host": v.cpu()}
    print("[host] parts", nds, B, flush=True)
    ref, at = [], 0
    for ds, c in zip(dss, per):
        if c:
            o, g, st = kf.scv([ds], v[at:at + c].clone(), status=True)
            a = kf.scv_adjoint([ds], v[at:at + c].clone(), go[at:at + c].clone())
            ref.append((o, g, a))
            assert not st.any()
        at += c
    for name, x in forms.items():
        o, g = kf.scv(dss, x, per_ds=per)
        assert torch.equal(o, torch.cat([r[0] for r in ref])), name
        assert torch.equal(g, torch.cat([r[1] for r in ref])), name
        a = kf.scv_adjoint(dss, x, go.expand(2, B)[1], per_ds=per)
        assert torch.equal(a, torch.cat([r[2] for r in ref])), name
    psi = kf.psi_batch(dss, [0.3 * np.eye(2)] * nds, 2)
    for j in (0, _lib.MAX_PSI_DS, nds - 1):
        assert torch.equal(psi[j], kf.psi_batch([dss[j]], [0.3 * np.eye(2)], 2)[0])


def test_side_stream():
    """The current stream is the one that the work goes to."""
    import paper_1511_07482_amd as kf
    rng = np.random.default_rng(6)
    X = torch.tensor(rng.standard_normal((500, 1)), device="cuda")
    v = torch.tensor([[0.4], [0.7]], dtype=torch.float64, device="cuda")
    want = kf.scv([kf.Dataset(X, np.eye(1) * 0.2, M=[64])], v)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        late = torch.zeros_like(v)
        for _ in range(50):
            late = late + v / 50          # the call must wait for these
        late.copy_(v)
        got = kf.scv([kf.Dataset(X, np.eye(1) * 0.2, M=[64])], late)
    side.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
