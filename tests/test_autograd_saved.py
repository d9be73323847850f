"""What torch's saved-tensor hooks hand back to fake_quantize's backward is looked at before its addresses
go to the library: the descriptor holds bare pointers, and the extents are those of the forward.  The checks
are host code, so the backward is called here with a context of our own and CPU tensors, up to the launch."""
import types

import pytest
import torch

from paper_2511_12653_amd import autograd
from paper_2511_12653_amd import binding as fq

import _gpu_harness as H


def _backward(monkeypatch, x, theta, gy, view=(2, 3, 8)):
    calls = []
    monkeypatch.setattr(autograd.fq, "fq_backward", lambda t, ws, stream=None: calls.append(t))
    ctx = types.SimpleNamespace(saved_tensors=(x, theta), needs_input_grad=(True, True) + (False,) * 6,
                                meta=(view, -127, 127, 0.0, fq.FLT_MIN, float("inf")))
    try:
        return autograd._FakeQuantize.backward(ctx, gy), calls
    except Exception:
        assert not calls
        raise


def test_what_the_forward_saved_is_accepted(monkeypatch):
    x, theta = torch.zeros(2, 3, 8), torch.zeros(3)
    (gx, gtheta, *rest), calls = _backward(monkeypatch, x, theta, torch.zeros_like(x))
    assert len(calls) == 1 and calls[0].x == x.data_ptr() and calls[0].gx == gx.data_ptr()
    assert gx.shape == x.shape and gtheta.shape == theta.shape and rest == [None] * 6


@pytest.mark.parametrize("name, x, theta, error", [
    ("x in other strides", torch.zeros(8, 3, 2).transpose(0, 2), torch.zeros(3), ValueError),
    ("x expanded", torch.zeros(1, 3, 8).expand(2, 3, 8), torch.zeros(3), ValueError),
    ("x with fewer elements", torch.zeros(2, 3, 7), torch.zeros(3), ValueError),
    ("x of another type than gy", torch.zeros(2, 3, 8, dtype=torch.float16), torch.zeros(3), TypeError),
    ("theta in 16 bits", torch.zeros(2, 3, 8), torch.zeros(3, dtype=torch.float16), TypeError),
    ("theta in 64 bits", torch.zeros(2, 3, 8), torch.zeros(3, dtype=torch.float64), TypeError),
    ("theta with fewer elements", torch.zeros(2, 3, 8), torch.zeros(2), ValueError),
])
def test_other_tensors_are_refused(monkeypatch, name, x, theta, error):
    gy = torch.zeros(x.shape)
    with pytest.raises(error):
        _backward(monkeypatch, x, theta, gy)


@pytest.mark.gpu
def test_hooks_that_move_the_saved_tensors():
    H.say("autograd: saved tensors to the host and back, then in other strides")
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((4, 6, 50), generator=gen, device="cuda", requires_grad=True)
    theta = torch.full((6,), -3.0, device="cuda", requires_grad=True)
    gy = torch.randn((4, 6, 50), generator=gen, device="cuda")
    run = lambda: autograd.fake_quantize(x, theta, -8, 7, channel_dim=1)
    want = torch.autograd.grad(run(), (x, theta), gy)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
        y = run()
    for a, b in zip(torch.autograd.grad(y, (x, theta), gy), want):
        assert torch.equal(a, b)
    twist = lambda t: t.transpose(0, 2).contiguous().transpose(0, 2) if t.dim() == 3 else t
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, twist):
        y = run()
    with pytest.raises(ValueError):
        torch.autograd.grad(y, (x, theta), gy)
