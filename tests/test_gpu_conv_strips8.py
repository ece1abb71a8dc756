"""The conv in strips of 8 tokens (bf16, four taps, from 80000 threads of 8 channels x 16 tokens up to 131072) and on both sides of that
range: last strips of 1 to 8 tokens, with and without the rows before the first.  Against the oracle on the inputs as stored."""
import pytest

from test_gpu_conv_runs import test_conv1d_causal_strips as _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,Hh,d,W,halo", [
    (1, 4992, 32, 64, 4, True), (1, 5003, 32, 64, 4, False), (16, 331, 32, 64, 4, True), (300, 17, 20, 64, 4, True), (2000, 9, 8, 64, 4, False),
    (700, 24, 6, 128, 4, True), (1, 8191, 32, 64, 4, True), (1, 5003, 32, 64, 3, True)])
def test_conv1d_causal_strips_of_8(oracle, B, T, Hh, d, W, halo):
    _check(oracle, "bf16", B, T, Hh, d, W, halo)
