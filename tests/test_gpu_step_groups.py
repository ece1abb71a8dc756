"""The decode step at group sizes around its passes of four query heads, one of them to a wave, against the oracle."""
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload

import helpers as H
from test_gpu_walk import _case, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("gate_scale,eps", [(1.0, 0.0), (0.5, 0.25)])
@pytest.mark.parametrize("B,Hq,Hkv,d", [(1, 1, 1, 64), (2, 6, 2, 64), (3, 4, 1, 128), (1, 5, 1, 64), (2, 14, 2, 128), (1, 8, 1, 128), (2, 9, 1, 64)])
def test_step(oracle, B, Hq, Hkv, d, gate_scale, eps, dtype):
    wl = Workload("step", B, 1, Hq, Hkv, d, 4, dtype)
    print("step", wl, gate_scale, eps, flush=True)
    args = _case(wl, seed=92)
    dt = H.tdtype(wl)
    q, k, v, g = (H.dev(a, dt) for a in args[:4])
    S, z = H.dev(args[4]), H.dev(args[5])
    o = torch.empty_like(q)
    lawcat.gla_step(H.desc_for(wl, gate_scale=gate_scale, eps=eps), q, k, v, g, S, z, o)
    torch.cuda.synchronize()
    _check(wl, {"o": H.host(o), "S": H.host(S), "z": H.host(z)}, oracle.gla_prefill(*args[:4], gate_scale, eps, *args[4:]), "step")
