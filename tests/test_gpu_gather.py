"""Channels whose units' sums are gathered by the channel's last unit: more than four units.

The unit counts sit where the gathering can go wrong: just above the exchange tree, around a whole
round of a wavefront's and of a block's threads, more than a block reads in one round, ragged last
chunks.  One channel and several, both dtypes.  Every launch is compared bit for bit with the two-launch
mode, which adds the same sums in the same order, and with the oracle (1e-5 of the binary64 sum, as
everywhere); the partial sums and slots must be back at zero after each.  With FQ_FLAG_NO_POLL the
gathering unit gives up at once, so that the units that arrive after it finish the channel."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import workloads
from paper_2511_12653_amd import binding as fq

import _gpu_harness as H

pytestmark = pytest.mark.gpu

CHUNK = {np.float16: 10240, np.float32: 5120}     # largest chunk of a block, in elements


@pytest.mark.parametrize("dtype, outer, channels, inner, waves", [
    (np.float32, 1, 1, 5 * 5120, 0),                # few units
    (np.float16, 1, 1, 65 * 1024 + 3, 0),           # around a wavefront's lanes
    (np.float32, 1, 1, 256 * 5120, 0),              # exactly a block's threads or fewer
    (np.float16, 1, 1, 257 * 10240 + 1, 0),
    (np.float16, 1, 1, 2100 * 10240 + 7, 0),        # more than eight sums per thread
    (np.float16, 7, 3, 10240 + 9, 0),               # several channels, two chunks per slab
    (np.float32, 5, 2, 1, 0),                       # one element per unit
    (np.float16, 5, 1500, 72, 1),                   # a wavefront per unit
    (np.float32, 65, 70, 30, 1),                    # its second round of lanes
    (np.float16, 257, 17, 9, 1),
    (np.float16, 2100, 2, 9, 1),                    # many rows of a wavefront's lanes
])
def test_gathered_sums(dtype, outer, channels, inner, waves):
    rng = np.random.Generator(np.random.Philox(outer * 1000 + channels))
    x = (rng.standard_normal((outer, channels, inner)) * 2).astype(dtype)
    theta = workloads.theta_for_scale(rng.uniform(0.02, 0.05, channels))
    gys = [rng.standard_normal(x.shape).astype(dtype) for _ in range(2)]
    gys[1][:, 0] = 0.0                              # a sum of zero has to be told from an absent one
    cases = [workloads.TensorCase("gather", x.shape, outer, channels, inner, -128, 127, x, theta, g) for g in gys]
    want, dcs = [], []
    for c in cases:
        two = H.DeviceCase(c, want_q=False, flags=fq.FQ_FLAG_TWO_PASS)
        info = fq.fq_layout(two.desc)
        assert info.units_per_channel > 4 and info.wave_units == waves
        ws = H.workspace_for(two.desc, fq.FQ_MODE_BACKWARD)
        fq.fq_backward(two.desc, ws)
        torch.cuda.synchronize()
        assert not bool(ws.any())
        s, active, _, _ = H.oracle_forward(c)
        H.check_backward(two, s, active, "gather/two launches")
        want.append([t.clone() for t in (two.gs, two.gtheta, two.gx)])
        dcs.append([H.DeviceCase(c, want_q=False, flags=f) for f in (0, fq.FQ_FLAG_NO_POLL)])
    H.say("gather: %dx%dx%d %s, %d units per channel, wave units %d" % (
        outer, channels, inner, np.dtype(dtype).name, info.units_per_channel, waves))
    ws = H.workspace_for(dcs[0][0].desc, fq.FQ_MODE_BACKWARD)
    for rep in range(12):
        dc, w = dcs[rep % 2][rep // 6], want[rep % 2]
        for t in (dc.gs, dc.gtheta):
            t.fill_(float("nan"))
        fq.fq_backward(dc.desc, ws)
        torch.cuda.synchronize()
        for got, ref in zip((dc.gs, dc.gtheta, dc.gx), w):
            assert torch.equal(got.view(torch.uint8), ref.view(torch.uint8)), rep
        assert not bool(ws.any()), "sums or slots left behind"
