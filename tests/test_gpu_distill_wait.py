"""The loss without its gradient in one launch, on both sides of the number of tiles (64) from which the block that adds the
tiles' sums waits before it looks for them: narrow and wide tiles, against the oracle, and replayed against the eager call."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import binding as fq

import _gpu_harness as H
from test_gpu_distill import _pair, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype, shape, tiles", [
    (np.float16, (1, 5, 64 * 64), 64), (np.float16, (1, 5, 64 * 64 + 1), 65), (np.float16, (13, 45, 704), 143),
    (np.float16, (2, 129, 8192), 256), (np.float16, (1, 7, 20352), 159), (np.float16, (3, 44, 5760), 135),
    (np.float32, (1, 5, 32 * 64), 64), (np.float32, (1, 5, 32 * 64 + 1), 65), (np.float32, (7, 45, 832), 182),
    (np.float32, (4, 65, 4096), 256), (np.float32, (15, 9, 576), 135),
])
def test_loss_alone(oracle, dtype, shape, tiles):
    a, b = _pair(shape[1] * 5 + shape[2], shape, dtype)
    _run(a, b, 0.6, oracle, want_grad=False, label="%d tiles" % tiles)
    da, db = H.dev(a), H.dev(b)
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    d = fq.FqDistill.from_torch(*shape, da, db, out, None, lam=0.6)
    assert fq.fq_distill_workspace_bytes(d) == -(-(tiles * 32 + 8) // 256) * 256
    ws = torch.full((fq.fq_distill_workspace_bytes(d) // 8,), float("nan"), dtype=torch.float64, device="cuda")
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            fq.fq_distill_loss(d, ws)
    for rep in range(4):
        da.mul_(1.0 - 0.05 * rep)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        fq.fq_distill_loss(d, ws)
        torch.cuda.synchronize()
        assert torch.equal(got, out) and bool(torch.isfinite(out).all()), rep
