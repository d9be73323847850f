"""One workspace for a backward whose sums are gathered and for distillation calls in between, zeroed once.  A
partial sum that is not zero reads as a unit that has arrived, so the distillation loss, whichever way it takes,
has to leave nothing behind: every word is looked at, and the gradients stay the same bit for bit."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import binding as fq

import _gpu_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name, shape, dtype, grad", [
    ("one launch", (1, 9, 3000), torch.float16, True), ("one launch, no gradient", (2, 40, 131), torch.float32, False),
    ("fused and a sum", (1, 3, 40000), torch.float16, True), ("fused and a sum, no gradient", (3, 5, 20001), torch.float32, False),
    ("two reads", (1, 530, 257), torch.float16, True), ("two reads, many tiles", (2, 520, 9000), torch.float32, True),
    ("statistics alone", (1, 530, 260), torch.float32, False), ("no elements", (0, 8, 16), torch.float16, True),
])
def test_distillation_leaves_a_workspace_zero(name, shape, dtype, grad):
    H.say("shared workspace: %s, %s %s" % (name, shape, dtype))
    gen = torch.Generator(device="cuda").manual_seed(shape[1])
    n = 300 * 5120 + 7                               # one scale, 301 units: gathered
    x, gy = (torch.randn(n, generator=gen, device="cuda") for _ in range(2))
    theta = torch.full((1,), -3.0, device="cuda")
    gx, gs, gth = torch.empty_like(x), torch.empty(1, device="cuda"), torch.empty(1, device="cuda")
    t = fq.FqTensor.from_torch(1, 1, n, -127, 127, x=x, theta=theta, gy=gy, gx=gx, gs=gs, gtheta=gth)
    assert fq.fq_layout(t).units_per_channel > 4
    a, b = ((torch.randn(shape, generator=gen, device="cuda") * 1.5).to(dtype) for _ in range(2))
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    d = fq.FqDistill.from_torch(*shape, a, b, out, torch.empty_like(a) if grad else None, lam=0.5)
    need = max(fq.fq_workspace_bytes(t, fq.FQ_MODE_BACKWARD), fq.fq_distill_workspace_bytes(d))
    ws = torch.zeros(need // 8, dtype=torch.int64, device="cuda")
    want = None
    for rep in range(4):
        gs.fill_(float("nan"))
        gth.fill_(float("nan"))
        fq.fq_backward(t, ws)
        torch.cuda.synchronize()
        got = [v.clone() for v in (gx, gs, gth)]
        want = want or got
        for v, w in zip(got, want):
            assert torch.equal(v.view(torch.uint8), w.view(torch.uint8)), rep
        assert not bool(ws.any())
        fq.fq_distill_loss(d, ws)
        torch.cuda.synchronize()
        assert not bool(ws.any()), "%d words left" % int((ws != 0).sum())
    assert bool(torch.isfinite(want[1]).all()) and float(want[1]) != 0.0
