"""One to four tokens that the int8 GEMM's launch quantises: row lengths on both sides of those from which a thread takes another unit of 8 values of
each token (4096, 8192, 12288 values), up to the longest such a launch takes, and shapes with a ring of three panels (3457 to 4096
channels of 4096 values and more), bit for bit against the two separate calls and the oracle."""
import numpy as np
import pytest

import test_gpu_w8a8_own_quant as own
from test_gpu_w8a8_own_quant import B  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("N,K", [(20, 4104), (36, 5440), (6180, 5448), (20, 8192), (20, 8200), (6160, 12296), (16, 16320), (3460, 4096), (4096, 4104), (3472, 8000)])
def test_rounds(B, orc, dtype, N, K):  # noqa: F811
    own.test_equals_separate_calls(B, orc, dtype, N, K)
