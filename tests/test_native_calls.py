"""The binding's native calls: the usual forms of the arguments go straight to the library, every other one and
every error through the Python form, with the same outcome."""
import ctypes
import inspect
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2511_12653_amd import binding as fq
from paper_2511_12653_amd import workloads

import _gpu_harness as H

CALLS = {"fq_forward": "(t, stream=None)", "fq_backward": "(t, workspace, stream=None)", "fq_plan_run": "(plan, stream=None)",
         "fq_plan_run_adam": "(plan, step, stream=None)", "fq_distill_loss": "(d, workspace, stream=None)",
         "fq_workspace_bytes": "(tensors, mode)"}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_signature_and_argument_errors(name):
    call = getattr(fq, name)
    assert str(inspect.signature(call)) == CALLS[name]
    for args, kw in (((), {}), ((1, 2, 3, 4, 5), {}), ((1,), {"nonsense": 2})):
        with pytest.raises(TypeError):
            call(*args, **kw)


def test_workspace_bytes_of_every_form():
    t = fq.FqTensor(3, 5, 70000, fq.FQ_F16, -8, 7, 0.0, fq.FLT_MIN, 1.0, 0, 4096, 4096, None, 4096, None, 4096, 4096)
    for mode in (fq.FQ_MODE_FORWARD, fq.FQ_MODE_BACKWARD):
        want = fq.fq_workspace_bytes([t], mode)
        assert want > 0
        assert fq.fq_workspace_bytes(t, mode) == fq.fq_workspace_bytes(tensors=t, mode=mode) == want
        assert fq.fq_workspace_bytes(fq.fq_tensor_array([t]), mode) == want

    class Derived(fq.FqTensor):
        pass

    assert fq.fq_workspace_bytes(Derived.from_buffer_copy(t), 2) == fq.fq_workspace_bytes(t, 2)
    t.dtype = 9
    assert fq.fq_workspace_bytes(t, 1) == 0 and fq.fq_workspace_bytes(t, 1 << 40) == 0
    with pytest.raises((TypeError, ctypes.ArgumentError)):
        fq.fq_workspace_bytes(t, "1")


OUT_OF_RANGE = r"""
import torch
from paper_2511_12653_amd import binding as fq
if fq._fqcall:
    fq._fqcall.streams(lambda device: 0, lambda: 0, torch.Tensor)      # no GPU: stand-ins for torch's lookups
fq._current_stream = lambda: 0
t = fq.FqTensor(2, 3, 1000, fq.FQ_F16, -8, 7, 0.0, fq.FLT_MIN, 1.0, 0, 4096, None, None, 4096, None, 4096, 4096)
d = fq.FqDistill(2, 3, 1000, fq.FQ_F16, 1.0, 1e-8, 1.0, 4096, 4096, None, 4096)
for call, desc, too_small, crooked in ((fq.fq_backward, t, -6, -5), (fq.fq_distill_loss, d, -6, -5)):
    for python_form in (False, True):                # keywords go through the Python form
        for workspace, status in (((1 << 70, 1 << 20), too_small), ((4104, -1), crooked), (((1 << 64) + 4104, 1 << 20), crooked),
                                  ((4104, (1 << 64) + 5), too_small), ((-8, 1 << 70), too_small)):
            try:
                call(desc, workspace=workspace) if python_form else call(desc, workspace)
            except fq.FqError as e:
                assert e.status == status, (call, workspace, e.status)
            else:
                raise AssertionError("accepted")
print("same outcome")
"""


def _root():
    return os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_workspace_numbers_out_of_range_mean_what_they_mean_to_ctypes():
    """A pointer or size with more than 64 bits, or a negative one, keeps its lower 64 bits (refused by the library
    where it says so), whichever form takes the call."""
    p = subprocess.run([sys.executable, "-c", OUT_OF_RANGE], cwd=_root(), stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True)
    assert p.returncode == 0 and "same outcome" in p.stdout, p.stdout


@pytest.mark.gpu
def test_forms_of_workspace_and_stream():
    H.say("native calls: forms of workspace and stream")
    rng = np.random.Generator(np.random.Philox(8))
    x = rng.standard_normal((2, 3, 30000)).astype(np.float32)
    case = workloads.TensorCase("calls", x.shape, 2, 3, 30000, -128, 127, x, workloads.theta_for_scale(np.full(3, 0.03)),
                                rng.standard_normal(x.shape).astype(np.float32))
    dc = H.DeviceCase(case, want_q=False)
    t = dc.desc
    ws = H.workspace_for(t, fq.FQ_MODE_BACKWARD)
    nbytes = ws.numel() * 4
    side = torch.cuda.Stream()

    class Derived(fq.FqTensor):
        pass

    def outputs(call, names):
        bufs = [getattr(dc, n) for n in names]
        for b in bufs:
            b.fill_(float("nan"))
        torch.cuda.synchronize()
        call()
        torch.cuda.synchronize()
        return [b.clone() for b in bufs]

    def current():
        with torch.cuda.stream(side):
            fq.fq_forward(t)
            fq.fq_backward(t, ws)

    fwd = [lambda: fq.fq_forward(t), lambda: fq.fq_forward(t, None), lambda: fq.fq_forward(t, stream=side),
           lambda: fq.fq_forward(t, side.cuda_stream), lambda: fq.fq_forward(t=t), lambda: fq.fq_forward(Derived.from_buffer_copy(t)), current]
    got = [outputs(f, ("y", "s")) for f in fwd]
    assert all(torch.equal(a, b) for g in got[1:] for a, b in zip(g, got[0])) and not bool(got[0][0].isnan().any())
    bwd = [lambda: fq.fq_backward(t, ws), lambda: fq.fq_backward(t, (ws.data_ptr(), nbytes)), lambda: fq.fq_backward(t, workspace=ws),
           lambda: fq.fq_backward(t, ws, side), lambda: fq.fq_backward(t, torch.nn.Parameter(ws, requires_grad=False)),
           lambda: fq.fq_backward(t, ws.view(torch.uint8)), lambda: fq.fq_backward(t, (ws.data_ptr() + (1 << 64), -1)), current]
    got = [outputs(f, ("gx", "gtheta")) for f in bwd]
    assert all(torch.equal(a, b) for g in got[1:] for a, b in zip(g, got[0])) and not bool(got[0][1].isnan().any())

    for bad in (None, (0, 0), (ws.data_ptr(), nbytes - 1), ws[:1], (ws.data_ptr() + 4, nbytes), (1 << 70, nbytes)):
        with pytest.raises(fq.FqError):
            fq.fq_backward(t, bad)
    with pytest.raises(fq.FqError) as e:
        fq.fq_forward(fq.FqTensor(1, 1, 8, 7, -8, 7))
    assert e.value.status == -2
    for bad in (None, 5, [t]):
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            fq.fq_forward(bad)

    table = H.workspace_for([t], fq.FQ_MODE_FORWARD)
    plan = fq.fq_plan_create([t], fq.FQ_MODE_FORWARD, table)
    want = outputs(lambda: fq.fq_plan_run(plan), ("y",))
    for f in (lambda: fq.fq_plan_run(plan, None), lambda: fq.fq_plan_run(plan=plan, stream=side), lambda: fq.fq_plan_run(plan.value),
              lambda: fq.fq_plan_run_adam(plan, 3), lambda: fq.fq_plan_run_adam(plan, np.int64(3))):
        assert torch.equal(outputs(f, ("y",))[0], want[0])
    with pytest.raises(fq.FqError):
        fq.fq_plan_run(ctypes.c_void_p())
    with pytest.raises(fq.FqError):
        fq.fq_plan_run_adam(plan, 0)
    fq.fq_plan_destroy(plan)
