"""Blocks of decode steps and fp32 prefill of a few tokens, on both sides of the change to the walk in chunks: group sizes around
its batches of four query heads, one part and several, with and without a start state, against the oracle."""
import pytest

from paper_2509_18467_amd.inputs import Workload

from test_gpu_walk import _case, _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 12, 13])
@pytest.mark.parametrize("call,dtype,start", [("prefill", "fp32", True), ("prefill", "fp32", False), ("steps", "fp32", True), ("steps", "bf16", True)])
@pytest.mark.parametrize("B,Hq,Hkv,d,gate_scale,eps", [(1, 1, 1, 64, 1.0, 0.0), (2, 6, 2, 64, 0.5, 0.0), (3, 16, 2, 64, 1.0, 0.25), (70, 16, 8, 64, 1.0, 0.0), (2, 3, 1, 128, 1.0, 0.0), (1, 16, 1, 128, 2.0, 0.0),
                                                       (1, 10, 2, 128, 1.0, 0.25), (40, 16, 1, 128, 0.5, 0.0)])
def test_a_few_tokens(oracle, B, Hq, Hkv, d, gate_scale, eps, call, dtype, start, T):
    wl = Workload("few", B, T, Hq, Hkv, d, 4, dtype)
    print("a few tokens", call, wl, gate_scale, eps, start, flush=True)
    args = _case(wl, seed=91)
    if not start:
        args = (*args[:4], None, None)
    _check(wl, _run(wl, call, *args, gate_scale=gate_scale, eps=eps), oracle.gla_prefill(*args[:4], gate_scale, eps, *args[4:]), f"few {call}")
