"""The lines of the backward's burst schedule for FP16: 769 to 1024 blocks of 900 vectors and more.  The checks are
those of test_gpu_chunk_rows (oracle, NaN in the edges, and the two-launch mode bit for bit)."""
import numpy as np
import pytest

from test_gpu_chunk_rows import test_rows_and_schedules as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels, vecs", [(768, 1025), (769, 899), (769, 900), (1024, 900), (1024, 1280), (1025, 900)])
@pytest.mark.parametrize("odd", [0, -1])
def test_lines(channels, vecs, odd):
    check(np.float16, channels, vecs, odd)
