"""The forward's block widths: 256 or 512 threads share a chunk, by the number of blocks and the vectors of a chunk.

Both sides of each line of the rule (blocks and vectors of a chunk are as listed, one vector more with `odd` elements more), whole vectors and slabs off the 16-byte grid, y, y with codes and codes alone,
in place, and one linear grid (more channels than a grid's y extent holds).  Against the oracle: y to 1 ulp, codes and
scales exactly."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import workloads
from paper_2511_12653_amd import binding as fq

import _gpu_harness as H

pytestmark = pytest.mark.gpu

N = {np.float16: 8, np.float32: 4}


@pytest.mark.parametrize("dtype, blocks, vecs", [
    (np.float16, 225, 512), (np.float32, 512, 256), (np.float16, 512, 257), (np.float32, 512, 512), (np.float16, 512, 513),
    (np.float32, 512, 1024), (np.float16, 512, 1025), (np.float16, 513, 1024), (np.float32, 513, 1025), (np.float32, 640, 1279),
    (np.float16, 641, 1279), (np.float32, 768, 1279), (np.float16, 769, 1279), (np.float16, 1799, 600), (np.float16, 1800, 448),
    (np.float32, 1800, 449), (np.float16, 1800, 513), (np.float32, 1801, 1025), (np.float16, 66000, 321),
])
@pytest.mark.parametrize("odd", [0, 3, -1])
def test_widths(dtype, blocks, vecs, odd):
    if blocks > 65535 and odd:
        return
    inner = vecs * N[dtype] + odd
    rng = np.random.Generator(np.random.Philox(blocks * 10000 + inner))
    x = (rng.standard_normal((1, blocks, min(inner, 700))) * 2).astype(dtype)
    x = np.ascontiguousarray(np.tile(x, (1, 1, -(-inner // x.shape[2])))[:, :, :inner])
    x[0, blocks // 2, 0] = np.nan
    x[0, blocks // 3, inner - 1] = np.inf
    theta = workloads.theta_for_scale(rng.uniform(0.02, 0.05, blocks))
    case = workloads.TensorCase("wide", x.shape, 1, blocks, inner, -128, 127, x, theta, None)
    ref = H.oracle_forward(case)
    for what in ("y", "inplace", "y and codes", "codes"):
        if blocks > 65535 and what != "y":
            continue
        H.say("forward width: %dx%d %s %s" % (blocks, inner, np.dtype(dtype).name, what))
        dc = H.DeviceCase(case, want_q="codes" in what, inplace=what == "inplace")
        cut = fq.fq_layout(dc.desc)
        assert (cut.blocks, -(-cut.unit_elems // N[dtype]), cut.wave_units) == (blocks, vecs + (odd > 0), 0)
        if what == "codes":
            dc.desc.y = None
        fq.fq_forward(dc.desc)
        torch.cuda.synchronize()
        if what != "codes":
            H.check_forward(dc, ref, "forward width")
        else:
            dc.check_guards("forward width")
            assert np.array_equal(dc.host("q").astype(np.int32), ref[3])
            assert np.array_equal(dc.host("s").view(np.uint32), ref[0].view(np.uint32))
