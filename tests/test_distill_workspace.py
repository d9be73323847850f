"""fq_distill_workspace_bytes: one workspace serves a pair with its gradient and without, at any alignment, whichever tiles the
two launches take."""
import random

import pytest

from paper_2511_12653_amd import binding as fq


def need(shape, dtype, grad, shift):
    at = 1 << 40
    size = 2 if dtype == fq.FQ_F16 else 4
    d = fq.FqDistill(*shape, dtype, 0.5, 1e-8, 1.0, at + shift * size, at + (1 << 38), at + (1 << 39) if grad else None, 1 << 20)
    return fq.fq_distill_workspace_bytes(d)


@pytest.mark.parametrize("dtype", [fq.FQ_F16, fq.FQ_F32], ids=["fp16", "fp32"])
def test_with_gradient_and_without(dtype):
    rng = random.Random(5)
    shapes = [(512, 256, 128), (513, 256, 128), (513, 160, 64), (700, 100, 127), (4, 180, 15730), (15, 249, 11944), (6, 101, 13352)]
    shapes += [(rng.randint(1, 16), rng.randint(8, 512), rng.choice([1, 2, 4, 64]) * rng.randint(30, 9000)) for _ in range(3000)]
    for shape in shapes:
        assert need(shape, dtype, True, 0) == need(shape, dtype, False, 0) > 0, shape
        if dtype == fq.FQ_F16 and shape[1] <= 256:
            assert need(shape, dtype, True, 1) == need(shape, dtype, False, 1) == need(shape, dtype, False, 0), shape
