"""The gathering by one wavefront, up to 256 units per channel, and the block-wide one beyond it.

Unit counts around one, two and four loads per lane and around the line between the two ways, as blocks and as
wavefronts.  gx goes out behind the unit's sum: into a buffer of its own, over gy (in place) and not at all.
Compared bit for bit with the two-launch mode and with the oracle (gx exact, sums to 1e-5, as everywhere)."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import workloads
from paper_2511_12653_amd import binding as fq

import _gpu_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gx", ["own", "inplace", "none"])
@pytest.mark.parametrize("dtype, units, channels, waves", [
    (np.float16, 5, 3, 0), (np.float32, 63, 3, 0), (np.float16, 64, 3, 0), (np.float32, 65, 3, 0),
    (np.float16, 129, 2, 0), (np.float32, 193, 2, 0), (np.float16, 255, 2, 0), (np.float32, 256, 2, 0),
    (np.float16, 257, 2, 0),
    (np.float16, 64, 257, 1), (np.float32, 65, 253, 1), (np.float16, 256, 65, 1), (np.float32, 257, 65, 1),
])
def test_one_wavefront_gathers(dtype, units, channels, waves, gx):
    rng = np.random.Generator(np.random.Philox(units * 100 + channels))
    shape = (units, channels, 75)
    x = (rng.standard_normal(shape) * 2).astype(dtype)
    gy = rng.standard_normal(shape).astype(dtype)
    theta = workloads.theta_for_scale(rng.uniform(0.02, 0.05, channels))
    case = workloads.TensorCase("edges", shape, units, channels, 75, -128, 127, x, theta, gy)
    H.say("gather edges: %d units, %d channels, %s, gx %s" % (units, channels, np.dtype(dtype).name, gx))
    s, active, _, _ = H.oracle_forward(case)
    got = []
    for extra in (0, fq.FQ_FLAG_NO_POLL, fq.FQ_FLAG_TWO_PASS):
        dc = H.DeviceCase(case, want_q=False, inplace=gx == "inplace", flags=extra | (fq.FQ_FLAG_NO_DX if gx == "none" else 0))
        info = fq.fq_layout(dc.desc)
        assert info.units_per_channel == units and info.wave_units == waves
        ws = H.workspace_for(dc.desc, fq.FQ_MODE_BACKWARD)
        fq.fq_backward(dc.desc, ws)
        torch.cuda.synchronize()
        assert not bool(ws.any()), "sums or slots left behind"
        H.check_backward(dc, s, active, "edges", want_gx=gx != "none")
        got.append((dc.gs, dc.gtheta))
    for other in got[:-1]:
        for a, b in zip(other, got[-1]):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
