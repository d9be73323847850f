"""Slabs that go one to a wavefront: in lists from 768 blocks of short slabs on, and in the forward of one tensor from 1024 blocks of at
most 192 vectors on.  Both sides of the lines, slabs off the 16-byte grid, a number of slabs that is no multiple of four
and members of a list that stay with blocks.  Against the oracle (bars as everywhere); lists also against the two-launch
mode of the same list, which adds the same sums in the same order, bit for bit.  At the line of the lists the cut shows in the
workspace; how a forward is cut shows nowhere, so there the results on both sides are all that is seen."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import binding as fq
from paper_2511_12653_amd import workloads

import _gpu_harness as H

pytestmark = pytest.mark.gpu


def _case(rng, outer, channels, inner, dtype):
    x = (rng.standard_normal((outer, channels, inner)) * 2).astype(dtype)
    gy = rng.standard_normal(x.shape).astype(dtype)
    return workloads.TensorCase("cut", x.shape, outer, channels, inner, -128, 127, x,
                                workloads.theta_for_scale(rng.uniform(0.02, 0.05, channels)), gy)


@pytest.mark.parametrize("what", ["y", "codes"])
@pytest.mark.parametrize("dtype, outer, channels, inner", [
    (np.float16, 1, 1023, 800), (np.float16, 1, 1024, 800), (np.float32, 3, 343, 768), (np.float32, 3, 343, 769),
    (np.float16, 2, 513, 1536), (np.float16, 2, 513, 1537), (np.float32, 1, 1025, 1), (np.float16, 5, 206, 49),
])
def test_forward_alone(dtype, outer, channels, inner, what):
    case = _case(np.random.Generator(np.random.Philox(channels + inner)), outer, channels, inner, dtype)
    H.say("wave cut forward: %dx%dx%d %s %s" % (outer, channels, inner, np.dtype(dtype).name, what))
    dc = H.DeviceCase(case, want_q=what == "codes")
    fq.fq_forward(dc.desc)
    torch.cuda.synchronize()
    H.check_forward(dc, None, "wave cut")


def _rounded(values):
    return -(-8 * values // 256) * 256


# units, channels: sums and slots of the list, where the cut shows in them.  Slabs of 2056 FP16 elements are two chunks each for blocks.
@pytest.mark.parametrize("shapes, units, channels", [
    ([(np.float16, 1, 64, 2056)] * 5 + [(np.float32, 1, 127, 49)], 5 * 128 + 127, 447),      # 767 blocks: two chunks per slab
    ([(np.float16, 1, 64, 2056)] * 6, 6 * 64, 384),                                          # 768: a wavefront per slab
    ([(np.float32, 1, 383, 49), (np.float16, 1, 384, 800)], 767, 767),
    ([(np.float32, 1, 384, 49), (np.float16, 1, 384, 800)], 768, 768),
    ([(np.float16, 4, 65, 1200), (np.float32, 1, 333, 147), (np.float16, 1, 3, 40000), (np.float32, 300, 1, 7)], 0, 0),
    ([(np.float32, 1, 384, 3456), (np.float32, 1, 128, 1152)], 768 + 256, 512),              # few short ones: blocks
    ([(np.float32, 1, 700, 319 * 4), (np.float32, 1, 70, 320 * 4), (np.float16, 70, 2, 9)], 0, 0),   # the longest slab, one more
])
def test_lists(shapes, units, channels):
    rng = np.random.Generator(np.random.Philox(len(shapes) * 31 + shapes[0][2]))
    cases = [_case(rng, o, c, k, d) for d, o, c, k in shapes]
    H.say("wave cut list: %s" % ([s[1:] for s in shapes],))
    dcs = [H.DeviceCase(c, want_q=False) for c in cases]
    descs = [d.desc for d in dcs]
    if units:
        beside_the_table = fq.fq_workspace_bytes(descs, fq.FQ_MODE_BACKWARD) - fq.fq_workspace_bytes(descs, fq.FQ_MODE_FORWARD)
        assert beside_the_table == _rounded(units) + _rounded(channels)
    ws = H.workspace_for(descs, fq.FQ_MODE_BACKWARD)
    for rep in range(2):
        fq.fq_multi_tensor(descs, fq.FQ_MODE_FORWARD, H.workspace_for(descs, fq.FQ_MODE_FORWARD))
        fq.fq_multi_tensor(descs, fq.FQ_MODE_BACKWARD, ws)
        torch.cuda.synchronize()
        for c, dc in zip(cases, dcs):
            ref = H.oracle_forward(c)
            H.check_forward(dc, ref, "wave cut list")
            H.check_backward(dc, ref[0], ref[1], "wave cut list")
    two = [H.DeviceCase(c, want_q=False, flags=fq.FQ_FLAG_TWO_PASS) for c in cases]
    descs = [d.desc for d in two]
    fq.fq_multi_tensor(descs, fq.FQ_MODE_BACKWARD, H.workspace_for(descs, fq.FQ_MODE_BACKWARD))
    torch.cuda.synchronize()
    for a, b in zip(dcs, two):
        for name in ("gx", "gs", "gtheta"):
            assert torch.equal(getattr(a, name).view(torch.uint8), getattr(b, name).view(torch.uint8))
