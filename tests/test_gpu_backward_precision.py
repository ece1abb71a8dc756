"""Rounding errors of the backward against 64 bits, no larger than those of the recurrence token by token in fp32."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload

import helpers as H

pytestmark = pytest.mark.gpu


def _library_alpha(g, gate_scale):
    """sigmoid(g)^gate_scale in fp32, one library function after the other."""
    g = H.dev(g)
    if gate_scale == 1.0:
        return H.host(1.0 / (1.0 + torch.exp2(-g * torch.tensor(1.44269504))))
    ls = torch.where(g < 0, g - torch.log1p(torch.exp(g)), -torch.log1p(torch.exp(-g)))
    return H.host(torch.exp(gate_scale * ls))


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("gate_scale", [1.0, 0.0625, 0.5, 2.0, 4.0])
@pytest.mark.parametrize("scale", [1.0, 4.0, 12.0])
def test_decay(gate_scale, scale, dtype):
    """One token, queries of one, denominators of one, dO of one in the first column: dS0's first column is alpha itself."""
    wl = Workload("decay", B=4, T=1, Hq=64, Hkv=64, d=64, dtype=dtype)
    print("decay", gate_scale, scale, dtype, flush=True)
    dt = H.tdtype(wl)
    g = (np.random.default_rng(71).standard_normal((wl.B, 1, 64, 64)) * scale).astype(np.float32)
    tg = H.dev(g, dt)
    g = H.host(tg).astype(np.float32)
    one, zero = torch.ones_like(tg), torch.zeros_like(tg)
    dO = torch.zeros_like(tg)
    dO[..., 0] = 1.0
    desc = H.desc_for(wl, gate_scale=gate_scale)
    outs = [torch.empty_like(tg) for _ in range(4)]
    dS0 = torch.empty(wl.B, 64, 64, 64, device="cuda")
    lawcat.gla_backward(desc, one, zero, zero, tg, torch.ones(wl.B, 1, 64, device="cuda"), dO, None, None, *outs, dS0, None,
                        lawcat.alloc_workspace(desc, lawcat.CALL_GLA_BACKWARD))
    torch.cuda.synchronize()
    ls = np.minimum(g, 0.0).astype(np.float64) - np.log1p(np.exp(-np.abs(g.astype(np.float64))))
    ref = np.exp(gate_scale * ls)
    keep = ref > 2.0 ** -126
    err = [np.sqrt(np.mean(((a - ref)[keep] / ref[keep]) ** 2)) * 2.0 ** 24 for a in (H.host(dS0)[:, None, :, :, 0], _library_alpha(g, gate_scale))]
    print(f"  RMS error {err[0]:.3f} units of 2^-24, with library functions {err[1]:.3f}", flush=True)
    # sixteen thousand values: either RMS is known to about one percent
    assert err[0] <= 1.02 * err[1]
