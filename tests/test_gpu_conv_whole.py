"""The conv's adjoint of two to four strips in all, one launch: sequences and strips of every number on both sides of it, lengths around
a strip and a run, channels that leave part of a workgroup idle, every width.  Against the oracle, the weights' gradient to 64 fp32
ulps of the sum of its terms' absolute values."""
import pytest

from test_gpu_conv_runs import test_conv1d_backward_runs as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,Hh,d,W", [
    (1, 65, 2, 64, 4), (1, 128, 1, 64, 4), (1, 129, 3, 128, 3), (1, 253, 2, 64, 2), (1, 256, 5, 64, 4), (1, 257, 2, 64, 4), (2, 5, 3, 64, 4),
    (2, 4, 3, 64, 4), (2, 67, 2, 64, 1), (3, 64, 1, 128, 4), (4, 7, 17, 64, 4), (4, 64, 2, 64, 3), (5, 33, 2, 64, 4), (2, 128, 32, 128, 4),
    (1, 65, 64, 128, 3), (1, 65, 65, 128, 4), (2, 33, 128, 128, 2), (2, 33, 129, 128, 1)])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_few_strips(oracle, dtype, B, T, Hh, d, W):
    check(oracle, dtype, B, T, Hh, d, W)
