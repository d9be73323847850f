"""The fused distillation kernel's long rows (256 bytes of a channel by 512 or 256 threads): both sides of the lines
that choose them (tiles per compute unit, the half-empty last tile, channels), every number of channels per lane,
ends of images, on the 4-element grid and off it, with and without a gradient.  Bars as in test_gpu_distill."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import binding as fq

from test_gpu_distill import _pair, _run

pytestmark = pytest.mark.gpu


def tiles_of(shape, dtype, misalign=0):
    """Tiles of a launch that a second kernel follows: its workspace is 16 bytes per tile, rounded up."""
    n, c, m = shape
    t = torch.empty(n * c * m + misalign, dtype=torch.float16 if dtype is np.float16 else torch.float32, device="cuda")[misalign:]
    out = torch.empty(3, dtype=torch.float64, device="cuda")
    return fq.fq_distill_workspace_bytes(fq.FqDistill.from_torch(n, c, m, t, t, out, None)) // 16


@pytest.mark.parametrize("dtype, shape, per_image", [
    # every number of channels per lane (512 full tiles of 128 / 64 positions); one channel more than the long rows hold
    *[(np.float16, (512, c, 128), 1) for c in (5, 17, 32, 33, 65, 97, 129, 193, 256)], (np.float16, (512, 257, 128), 2),
    *[(np.float32, (512, c, 64), 1) for c in (5, 33, 64, 65, 129, 193, 256)],
    # tiles per compute unit: seven eighths of the last round and one tile less, enough of them
    (np.float16, (448, 70, 128), 1), (np.float16, (447, 70, 128), 2), (np.float16, (1024, 70, 128), 1),
    (np.float16, (600, 9, 128), 1), (np.float16, (300, 9, 128), 2),
    # the last tile of an image half empty; few channels take it
    (np.float16, (512, 70, 129), 3), (np.float32, (500, 70, 129), 3), (np.float16, (512, 9, 260), 3), (np.float32, (500, 9, 132), 3),
    (np.float16, (30, 40, 2111), 17), (np.float32, (30, 40, 1090), 18),
    # off the grid
    (np.float16, (512, 33, 127), 1), (np.float16, (512, 9, 125), 1), (np.float32, (512, 40, 63), 1), (np.float32, (512, 9, 61), 1),
    (np.float32, (512, 129, 63), 1), (np.float32, (512, 100, 63), 1),
])
def test_long_rows(oracle, dtype, shape, per_image):
    wide = 128 if dtype is np.float16 else 64
    assert per_image in (-(-shape[2] // wide), -(-2 * shape[2] // wide))
    assert tiles_of(shape, dtype) == -(-shape[0] * per_image // 16) * 16
    a, b = _pair(shape[1] * 3 + shape[2], shape, dtype)
    _run(a, b, 0.6, oracle, upstream=64.0, label="long")
    if shape[1] in (9, 33, 70):
        _run(a, b, 0.6, oracle, want_grad=False, label="long")
        _run(a, b, 0.6, oracle, inplace="student", label="long")
