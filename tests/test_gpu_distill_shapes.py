"""The lines beyond which rows of 256 bytes go to 1024 threads or back to rows of 128: FP16 with 97 to 256 channels (whole cache
lines, images of an odd number of positions, with a gradient and without), FP32 with 193 to 256 channels and no gradient, and FP32 rows
that are no whole number of 64-byte halves of a line in launches of many elements.  Bars as in test_gpu_distill."""
import numpy as np
import pytest

from test_gpu_distill import _pair, _run
from test_gpu_distill_long import tiles_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype, shape, per_image", [
    # whole cache lines: two tiles to a compute unit and one more
    (np.float16, (512, 129, 128), 1), (np.float16, (513, 129, 128), 2), (np.float16, (513, 192, 128), 2),
    (np.float16, (513, 193, 128), 2), (np.float16, (513, 256, 128), 2), (np.float16, (1024, 128, 128), 1),
    # on the grid, off it
    (np.float16, (512, 129, 124), 1), (np.float16, (512, 200, 124), 1), (np.float16, (512, 150, 127), 1),
    # an odd number of positions: 97 to 128 channels and 193 to 256, six tiles to a compute unit and one less
    (np.float16, (512, 97, 127), 2), (np.float16, (1535, 128, 125), 2), (np.float16, (1536, 97, 126), 1),
    (np.float16, (512, 193, 127), 2), (np.float16, (1536, 193, 125), 1),
    (np.float32, (512, 193, 64), 1), (np.float32, (512, 256, 60), 1), (np.float32, (512, 256, 63), 1), (np.float32, (512, 192, 64), 1),
    # the same with a gradient and fewer than two tiles to a compute unit: 129 to 160 channels, and more in images of up to 56 tiles
    # (or 57); on the grid; two to each
    (np.float16, (4, 150, 14527), 227), (np.float16, (9, 161, 7167), 112), (np.float16, (8, 161, 7169), 57),
    (np.float16, (9, 161, 7164), 56), (np.float16, (512, 150, 125), 1),
    # 14 million elements with 57 to 64 channels, and with 56
    (np.float32, (3, 64, 72911), 1140), (np.float32, (3, 64, 72929), 1140), (np.float32, (3, 57, 81931), 1281),
    (np.float32, (3, 56, 83999), 1313),
    # 6.4 million elements
    (np.float32, (16, 100, 3996), 63), (np.float32, (16, 100, 4004), 63), (np.float32, (16, 200, 2004), 32),
])
def test_both_sides(oracle, dtype, shape, per_image):
    assert tiles_of(shape, dtype) == -(-shape[0] * per_image // 16) * 16
    a, b = _pair(shape[1] * 3 + shape[2], shape, dtype)
    _run(a, b, 0.6, oracle, upstream=64.0, label="shapes")
    _run(a, b, 0.6, oracle, want_grad=False, label="shapes")
