"""The conv's adjoint for batches of short sequences, on both sides of the changes between one, four and sixteen runs per strip, and
sums of dw over few partial sums and many.  Against the oracle on the inputs as stored."""
import pytest

from test_gpu_conv_runs import test_conv1d_backward_runs as _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,Hh,d,W", [
    # one thread per strip: 2^20 bytes of channels x sequences and more; the sequences shorter and as long as a strip
    (257, 1, 32, 64, 4), (257, 5, 32, 64, 4), (260, 17, 32, 64, 3), (129, 63, 32, 128, 4), (129, 64, 32, 128, 2), (300, 16, 7, 128, 4),
    # four, and sixteen
    (49, 9, 32, 64, 4), (47, 9, 32, 64, 4), (100, 4, 3, 64, 4), (100, 5, 3, 64, 4), (20, 64, 77, 64, 1),
    # 2, 16 and 17 partial sums
    (2, 3, 1, 64, 4), (16, 7, 3, 64, 4), (17, 7, 3, 64, 4)])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_conv1d_backward_short(oracle, dtype, B, T, Hh, d, W):
    _check(oracle, dtype, B, T, Hh, d, W)
