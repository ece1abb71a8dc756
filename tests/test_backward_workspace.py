"""The workspace of lawcat_gla_backward: its size for every length, and that the call stays within it."""
import numpy as np
import pytest

from paper_2509_18467_amd import lawcat


def _words(B, T, Hq, Hkv, d):
    """The size that callers may have kept: a word per token and query head, one per token, kv head and channel, two states and
    a row per segment (of a multiple of 64 tokens, about 1024 over all heads)."""
    heads = B * Hkv
    want = max(1, 1024 // heads)
    seg_len = -(-(-(-T // want)) // 64) * 64
    nseg = -(-T // seg_len)
    return B * T * Hq + B * T * Hkv * d + 2 * heads * nseg * (d * d + 2 * d) + heads * nseg * d


@pytest.mark.parametrize("dtype", [lawcat.DTYPE_BF16, lawcat.DTYPE_F32])
@pytest.mark.parametrize("B,Hq,Hkv,d", [(1, 1, 1, 64), (1, 32, 8, 64), (1, 32, 8, 128), (2, 6, 2, 64), (4, 32, 1, 64), (3, 16, 1, 128), (32, 32, 8, 64), (128, 32, 8, 64), (129, 8, 8, 128)])
def test_size(B, Hq, Hkv, d, dtype):
    for T in [*range(1, 80), 300, 1000, 1023, 1025, 2048, 5003, 16384, 20000, 32767, 32768, 131072, 131073]:
        need = lawcat.workspace_bytes(lawcat.make_desc(B, T, Hq, Hkv, d, dtype=dtype), lawcat.CALL_GLA_BACKWARD)
        assert 0 < need <= 4 * _words(B, T, Hq, Hkv, d) + 256, (T, need)


@pytest.mark.gpu
@pytest.mark.parametrize("T", [1, 15, 16, 17, 63, 65, 321, 1029])
@pytest.mark.parametrize("Hq,Hkv,d,dtype", [(6, 2, 64, "bf16"), (8, 2, 64, "bf16"), (3, 3, 64, "fp32"), (4, 1, 128, "fp32"), (2, 1, 128, "bf16")])
def test_the_call_stays_within(oracle, Hq, Hkv, d, dtype, T):
    import torch

    import helpers as H
    from paper_2509_18467_amd.inputs import Workload, make_inputs, round_to_bf16

    wl = Workload("workspace", B=2, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=dtype)
    print("workspace", wl, flush=True)
    x = make_inputs(wl, seed=81, state=True)
    rnd = round_to_bf16 if dtype == "bf16" else (lambda a: a)
    q, k = (rnd((np.abs(x[n]) + 0.05).astype(np.float32)) for n in ("Q", "K"))
    v, g, S0, z0 = x["V"], x["G"], x["S0"], np.abs(x["z0"]) + 0.5
    dO = rnd((np.random.default_rng(82).standard_normal(q.shape) * 0.5).astype(np.float32))
    den = oracle.gla_prefill(q, k, v, g, 0.25, 0.0, S0, z0)["den"].astype(np.float32)
    ref = oracle.gla_backward(q, k, v, g, dO, 0.25, 0.0, S0, z0)
    dt = H.tdtype(wl)
    desc = H.desc_for(wl, gate_scale=0.25)
    ins = [H.dev(a, dt) for a in (q, k, v, g)]
    outs = [torch.empty_like(t) for t in ins] + [torch.empty(2, Hkv, d, d, device="cuda"), torch.empty(2, Hkv, d, device="cuda")]
    need = lawcat.workspace_bytes(desc, lawcat.CALL_GLA_BACKWARD)
    # NaNs in the workspace: what the call reads of it, it has written; and a page behind it that it leaves alone
    ws = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    lawcat.gla_backward(desc, *ins, H.dev(den), H.dev(dO, dt), H.dev(S0), H.dev(z0), *outs, ws[:need])
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xFF).all())
    for n, t in zip(("dq", "dk", "dv", "dg", "dS0", "dz0"), outs):
        H.assert_close(H.host(t), ref[n], wl, f"workspace {n}", 1 if dtype == "bf16" and t.dtype == dt else 0)
