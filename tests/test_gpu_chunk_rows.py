"""Single-tensor launches on both sides of the lines that choose a kernel: the number of vectors a lane
has in a whole chunk (one to five, a kernel for each), and the backward's burst schedule (769 to 1024 blocks
of 900 vectors or more for FP16, 400 to 768 of 600 or more for FP32).  Slabs are a whole
number of vectors, or start off the 16-byte grid so that elements before and behind the vectors are left;
one slab has a NaN in such an element.  Against the oracle, bars as everywhere; the burst and the
interleaved schedule are also compared with the two-launch mode bit for bit."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import workloads
from paper_2511_12653_amd import binding as fq

import _gpu_harness as H

pytestmark = pytest.mark.gpu

N = {np.float16: 8, np.float32: 4}


@pytest.mark.parametrize("dtype, channels, vecs", [
    (np.float16, 769, 900), (np.float16, 768, 900), (np.float16, 769, 899), (np.float16, 768, 1280),
    (np.float16, 769, 1280), (np.float16, 70, 1025), (np.float16, 70, 1024), (np.float16, 70, 768),
    (np.float16, 70, 512), (np.float16, 70, 257), (np.float16, 70, 1),
    (np.float32, 400, 600), (np.float32, 399, 600), (np.float32, 400, 599), (np.float32, 768, 600), (np.float32, 769, 600), (np.float32, 500, 769),
    (np.float32, 768, 1025), (np.float32, 70, 1025), (np.float32, 70, 769), (np.float32, 70, 512), (np.float32, 70, 256),
])
@pytest.mark.parametrize("odd", [0, 1, -1])
def test_rows_and_schedules(dtype, channels, vecs, odd):
    inner = vecs * N[dtype] + odd
    rng = np.random.Generator(np.random.Philox(channels * 10000 + inner))
    x = (rng.standard_normal((1, channels, inner)) * 2).astype(dtype)
    if odd:
        x[0, channels // 2, 0] = np.nan
        x[0, channels // 3, inner - 1] = np.nan
    gy = rng.standard_normal(x.shape).astype(dtype)
    theta = workloads.theta_for_scale(rng.uniform(0.02, 0.05, channels))
    case = workloads.TensorCase("rows", x.shape, 1, channels, inner, -128, 127, x, theta, gy)
    H.say("rows: %dx%d %s" % (channels, inner, np.dtype(dtype).name))
    got = {}
    for flags in (0, fq.FQ_FLAG_TWO_PASS):
        dc = H.DeviceCase(case, want_q=False, flags=flags)
        if not flags:
            fq.fq_forward(dc.desc)
        fq.fq_backward(dc.desc, H.workspace_for(dc.desc, fq.FQ_MODE_BACKWARD))
        torch.cuda.synchronize()
        if not flags:
            ref = H.oracle_forward(case)
            s, active, y, _ = ref
            dc.check_guards("rows")
            assert H.ulp_distance(dc.host("y"), y).max() <= 1
            r = H.oracle_backward(case, s, active)
            assert np.array_equal(dc.host("gx").view(np.uint8), r["gx"].reshape(-1).view(np.uint8))
            bad = np.isnan(r["acc"])
            assert bad.sum() == (2 if odd and channels // 2 != channels // 3 else 0)
            for name, want in (("gs", r["acc"]), ("gtheta", r["gtheta"])):
                v = dc.host(name).astype(np.float64)
                assert np.array_equal(np.isnan(v), bad)
                assert np.all(np.abs(v - want)[~bad] <= H.GS_RTOL * np.abs(want)[~bad])
        got[flags] = (dc.host("gs"), dc.host("gtheta"), dc.host("gx"))
    for a, b in zip(got[0], got[fq.FQ_FLAG_TWO_PASS]):
        assert np.array_equal(a, b, equal_nan=True)
