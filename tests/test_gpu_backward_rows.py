"""The backward in bf16 storage around the ends of its chunks: rows that all threads of a workgroup load together, for one, two and four
query heads a pass and two passes, and products in bf16 terms; against the oracle at the bars of test_gpu_backward.py (2e-2 of RMS and
a half-ulp of the stored value; dS0 without that)."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload, make_inputs, round_to_bf16

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 4, 8])
@pytest.mark.parametrize("T", [1, 15, 16, 17, 70])
def test_chunk_ends(oracle, T, group, d):
    wl = Workload("rows", B=2, T=T, Hq=2 * group, Hkv=2, d=d, dtype="bf16")
    print("rows", wl, flush=True)
    x = make_inputs(wl, seed=23, state=True)
    q = round_to_bf16(np.float32(oracle.conv1d_causal(x["Q"], x["wq"], None, 1)))
    k = round_to_bf16(np.float32(oracle.conv1d_causal(x["K"], x["wk"], None, 1)))
    v, g, S0, z0 = x["V"], x["G"], x["S0"], x["z0"]
    fwd = oracle.gla_prefill(q, k, v, g, 0.5, 0.0, S0, z0)
    den = fwd["den"].astype(np.float32)
    dO = round_to_bf16(np.random.default_rng(6).standard_normal(fwd["o"].shape).astype(np.float32))
    ref = oracle.gla_backward(q, k, v, g, dO, 0.5, 0.0, S0, z0)
    desc = H.desc_for(wl, gate_scale=0.5)
    tq, tk, tv, tg, tO = (H.dev(a, H.tdtype(wl)) for a in (q, k, v, g, dO))
    out = {"dq": torch.empty_like(tq), "dk": torch.empty_like(tk), "dv": torch.empty_like(tv), "dg": torch.empty_like(tg),
           "dS0": torch.empty(wl.B, wl.Hkv, d, d, device="cuda")}
    lawcat.gla_backward(desc, tq, tk, tv, tg, H.dev(den), tO, H.dev(S0), H.dev(z0), out["dq"], out["dk"], out["dv"], out["dg"],
                        out["dS0"], None, lawcat.alloc_workspace(desc, lawcat.CALL_GLA_BACKWARD))
    torch.cuda.synchronize()
    for n, t in out.items():
        H.assert_close(H.host(t), ref[n], wl, f"rows {n}", 0 if n == "dS0" else 1)
