"""Lists on both sides of what a wavefront's lanes look through at once (64 tensors), empty members among
them, and the Adam steps of a plan: the bias corrections that ride along with a launch where all betas are the
same, the copied table where they are not, and what fq_plan_run, eager or captured, sees afterwards."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import workloads
from paper_2511_12653_amd import binding as fq

import _gpu_harness as H

pytestmark = pytest.mark.gpu


def _case(rng, outer, channels, inner, dtype):
    x = (rng.standard_normal((outer, channels, inner)) * 2).astype(dtype)
    gy = rng.standard_normal(x.shape).astype(dtype)
    theta = workloads.theta_for_scale(rng.uniform(0.02, 0.05, channels))
    return workloads.TensorCase("t", x.shape, outer, channels, inner, -128, 127, x, theta, gy)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129, 200])
def test_every_block_finds_its_tensor(n):
    rng = np.random.Generator(np.random.Philox(n))
    cases = []
    for i in range(n):
        dtype = np.float16 if rng.integers(0, 2) else np.float32
        empty = i % 7 == 3
        cases.append(_case(rng, 0 if empty else int(rng.integers(1, 7)), int(rng.integers(1, 12)),
                           int(rng.choice([1, 30, 257, 2100])), dtype))
    H.say("lookup: %d tensors" % n)
    dcs = [H.DeviceCase(c, want_q=False) for c in cases]
    arr = fq.fq_tensor_array([d.desc for d in dcs])
    for mode in (fq.FQ_MODE_FORWARD, fq.FQ_MODE_BACKWARD):
        fq.fq_multi_tensor(arr, mode, H.workspace_for(arr, mode))
    torch.cuda.synchronize()
    for i, (c, d) in enumerate(zip(cases, dcs)):
        if c.numel:
            ref = H.oracle_forward(c)
            H.check_forward(d, ref, "lookup[%d of %d]" % (i, n))
            H.check_backward(d, ref[0], ref[1], "lookup[%d of %d]" % (i, n))


@pytest.mark.parametrize("n, channels, inner, dtype", [
    # theta in front of the rows or behind: up to 768 blocks, more of them with whole chunks, more with short ones
    (3, 256, 5120, np.float32), (4, 200, 5120, np.float32), (4, 200, 10240, np.float16), (5, 200, 2400, np.float16),
])
def test_lists_with_codes(n, channels, inner, dtype):
    rng = np.random.Generator(np.random.Philox(n * channels))
    cases = [_case(rng, 1, channels, inner, dtype) for _ in range(n)] + [_case(rng, 2, 3, 77, dtype)]
    H.say("list with codes: %d x (1, %d, %d) %s" % (n, channels, inner, np.dtype(dtype).name))
    dcs = [H.DeviceCase(c, want_q=i % 2 == 0) for i, c in enumerate(cases)]
    arr = fq.fq_tensor_array([d.desc for d in dcs])
    fq.fq_multi_tensor(arr, fq.FQ_MODE_FORWARD, H.workspace_for(arr, fq.FQ_MODE_FORWARD))
    torch.cuda.synchronize()
    for i, (c, d) in enumerate(zip(cases, dcs)):
        H.check_forward(d, H.oracle_forward(c), "codes[%d]" % i)


@pytest.mark.parametrize("same", [True, False])
def test_adam_steps_of_a_plan(same):
    rng = np.random.Generator(np.random.Philox(99))
    cases = [_case(rng, 2, 5, 700, np.float32), _case(rng, 1, 3, 9000, np.float16), _case(rng, 9, 4, 64, np.float32)]
    betas = [(0.9, 0.999)] * 3 if same else [(0.9, 0.999), (0.8, 0.99), (0.9, 0.999)]
    H.say("plan adam: same betas %s" % same)

    def fresh():
        dcs = [H.DeviceCase(c, want_q=False) for c in cases]
        state = [(torch.zeros(c.channels, device="cuda"), torch.zeros(c.channels, device="cuda")) for c in cases]
        return dcs, state

    def adam(k, dc, st, step):
        return fq.FqAdam.from_torch(st[0], st[1], dc.theta, lr=1e-2, beta1=betas[k][0], beta2=betas[k][1], step=step)

    # one tensor at a time, the step in the descriptor
    steps = [1, 2, 3, 3, 7, 7, 7, 8]
    one, ostate = fresh()
    wss = [H.workspace_for(d.desc, fq.FQ_MODE_BACKWARD) for d in one]
    for step in steps:
        for k, (d, st, ws) in enumerate(zip(one, ostate, wss)):
            d.desc.set_adam(adam(k, d, st, step))
            fq.fq_backward(d.desc, ws)
    # the plan: 1, 2, 3, then whatever is in place (eager), 7, twice what is in place (captured), 8
    dcs, state = fresh()
    for k, (d, st) in enumerate(zip(dcs, state)):
        d.desc.set_adam(adam(k, d, st, 1))
    arr = fq.fq_tensor_array([d.desc for d in dcs])
    ws = H.workspace_for(arr, fq.FQ_MODE_BACKWARD)
    plan = fq.fq_plan_create(arr, fq.FQ_MODE_BACKWARD, ws)
    try:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fq.fq_plan_run(plan)
        for step in (1, 2, 3):
            fq.fq_plan_run_adam(plan, step)
        fq.fq_plan_run(plan)
        fq.fq_plan_run_adam(plan, 7)
        graph.replay()
        graph.replay()
        fq.fq_plan_run_adam(plan, 8)
        torch.cuda.synchronize()
    finally:
        fq.fq_plan_destroy(plan)
    for k in range(3):
        for a, b in ((one[k].theta, dcs[k].theta), (ostate[k][0], state[k][0]), (ostate[k][1], state[k][1])):
            # sums in another order reach theta through a gradient rounded once to binary32
            np.testing.assert_allclose(a.cpu().numpy(), b.cpu().numpy(), rtol=1e-5, atol=1e-9)
