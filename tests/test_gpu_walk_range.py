"""The walk in chunks over fp32's range: without eps an output does not depend on the scale of its query, down to where the
products of a query with the normalizer leave fp32."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd.inputs import Workload

import helpers as H
from test_gpu_walk import _case, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("power", [-90, -70, 70])
@pytest.mark.parametrize("call,dtype,d,Hq", [("prefill", "fp32", 64, 4), ("steps", "fp32", 128, 2), ("steps", "bf16", 64, 8), ("prefill", "fp32", 128, 6)])
def test_scale_of_the_queries(call, dtype, d, Hq, power):
    wl = Workload("range", 1, 45, Hq, 2, d, 4, dtype)
    print("walk, scaled queries", call, wl, power, flush=True)
    q, k, v, g, S0, z0 = _case(wl, 95)
    g[:, :, 0] = H.host(torch.tensor(-2.6875))      # a chunk decays by nearly 2^-64
    a = _run(wl, call, q, k, v, g, S0, z0)
    b = _run(wl, call, q * np.float32(2.0) ** np.float32(power), k, v, g, S0, z0)
    for n in ("o", "S", "z"):
        assert np.array_equal(a[n], b[n]), n
