"""A call goes to the current stream: its input is written there behind
milliseconds of other work, so that a launch on any other stream would read
what was there before."""
import numpy as np
import pytest
import torch

from _gpu_util import log

pytestmark = pytest.mark.gpu


def test_call_waits_for_its_stream(kf, gpu):
    rng = np.random.default_rng(6)
    X = torch.tensor(rng.standard_normal((500, 1)), device=gpu)
    v = torch.tensor([[0.4], [0.7]], dtype=torch.float64, device=gpu)
    ds = kf.Dataset(X, np.eye(1) * 0.2, M=[64])
    want = kf.scv([ds], v)
    old = kf.scv([ds], torch.ones_like(v))
    assert not torch.equal(want[0], old[0])
    big = torch.ones(4096, 4096, device=gpu)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.mm(big, big)   # (the library's own set-up)
        late = torch.ones_like(v)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(side):
        for _ in range(40):
            torch.mm(big, big)
        late.copy_(v)
        done.record()
        got = kf.scv([ds], late)
        waiting = not done.query()   # the input was still to be written when the call returned
    side.synchronize()
    log(f"[stream] input pending at the call: {waiting}")
    assert waiting
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
