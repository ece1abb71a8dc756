"""fp32 prefill cut into segments: lengths around the segments' tokens, one to eight segments, against the oracle; no further from it
than the walk in one piece; without the workspace (or with too little of it, or in place) that walk, bit for bit; tokens that are not
finite spoil the same outputs."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu


def _call(x, wl, ws, state=True, gate_scale=1.0, carry=0, short=0):
    D = lawcat.make_desc(wl.B, wl.T, wl.Hq, wl.Hkv, wl.d, dtype=lawcat.DTYPE_F32, gate_scale=gate_scale, carry_mode=carry)
    q, k, v, g = (H.dev(x[n]) for n in ("Q", "K", "V", "G"))
    S0, z0 = (H.dev(x["S0"]), H.dev(x["z0"])) if state else (None, None)
    o, den = torch.empty_like(q), torch.empty(wl.B, wl.T, wl.Hq, device="cuda")
    S, z = torch.empty(wl.B, wl.Hkv, wl.d, wl.d, device="cuda"), torch.empty(wl.B, wl.Hkv, wl.d, device="cuda")
    need = lawcat.workspace_bytes(D, lawcat.CALL_GLA_PREFILL)
    buf = torch.full((need + 256,), 0x5A, dtype=torch.uint8, device="cuda") if ws else None
    lawcat.gla_prefill(D, q, k, v, g, S0, z0, o, den, S, z, buf[:need - short] if need and ws else None)
    torch.cuda.synchronize()
    if ws:
        assert bool((buf[need:] == 0x5A).all())
    return {"o": H.host(o), "den": H.host(den), "S": H.host(S), "z": H.host(z)}, need


def _inputs(wl, seed):
    x = make_inputs(wl, seed=seed, state=True)
    for n in ("Q", "K"):
        x[n] = np.where(x[n] > 0, 1 + x[n], np.exp(x[n])).astype(np.float32)
    return x


@pytest.mark.parametrize("d,Hq,Hkv,B,T,gate_scale", [
    (64, 2, 2, 1, 64, 1.0), (64, 2, 2, 1, 63, 1.0), (64, 2, 2, 1, 65, 0.0625), (64, 2, 2, 1, 256, 1.0), (64, 4, 2, 1, 257, 0.0625), (64, 8, 2, 2, 511, 1.0),
    (64, 64, 16, 4, 200, 0.25), (128, 2, 2, 1, 96, 1.0), (128, 2, 2, 1, 95, 1.0), (128, 8, 2, 2, 289, 0.0625), (128, 32, 8, 3, 130, 1.0)])
def test_segments(oracle, d, Hq, Hkv, B, T, gate_scale):
    wl = Workload("segments", B, T, Hq, Hkv, d, 4, "fp32")
    x = _inputs(wl, 91)
    print("walk segments", wl, flush=True)
    got, need = _call(x, wl, 1, gate_scale=gate_scale)
    assert (need > 0) == (T >= (64 if d == 64 else 96))
    whole, _ = _call(x, wl, 0, gate_scale=gate_scale)
    ref = oracle.gla_prefill(x["Q"], x["K"], x["V"], x["G"], gate_scale, 0.0, x["S0"], x["z0"])
    for n in ("o", "den", "S", "z"):
        H.assert_close(got[n], ref[n], wl, n)
        # fewer roundings than the whole walk, but others: within a thirty-second of an ulp of its error
        e, w = (np.linalg.norm(a[n] - ref[n]) / np.linalg.norm(ref[n]) for a in (got, whole))
        assert e <= w + 2.0 ** -29, (n, e, w)


def test_without_the_workspace():
    wl = Workload("segments", 1, 256, 4, 2, 64, 4, "fp32")
    x = _inputs(wl, 92)
    whole, need = _call(x, wl, 0)
    assert need > 0
    small, _ = _call(x, wl, 1, short=16)
    for n in whole:
        assert np.array_equal(whole[n], small[n])
    serial, none = _call(x, wl, 1, carry=lawcat.CARRY_SEQUENTIAL)
    assert none == 0
    for n in whole:
        assert np.array_equal(whole[n], serial[n])


@pytest.mark.parametrize("what,value", [("K", np.inf), ("V", np.inf), ("V", np.nan), ("Q", np.nan), ("K", 3e37)])
def test_tokens_that_are_not_finite(what, value):
    wl = Workload("segments", 1, 256, 2, 2, 64, 4, "fp32")
    x = _inputs(wl, 93)
    x[what][0, 100, 0, 5] = value
    got, _ = _call(x, wl, 1)
    whole, _ = _call(x, wl, 0)
    for n in got:
        assert np.array_equal(np.isfinite(got[n]), np.isfinite(whole[n])), n
    assert np.isfinite(got["o"][0, :100]).all()


def test_the_feature_map_layer_whatever_the_workspace():
    """lawcat_layer_prefill_fm in fp32 storage asks for no segments' workspace: more than it asks for changes no bit."""
    wl = Workload("segments", 1, 300, 4, 2, 64, 4, "fp32")
    x = make_inputs(wl, seed=94)
    wf = np.stack([np.eye(64, dtype=np.float32)] * 2)
    D = H.desc_for(wl, feature_map=1, gate_scale=0.0625)
    Q, K, V, G, wq, wk = (H.dev(x[n]) for n in ("Q", "K", "V", "G", "wq", "wk"))
    need = lawcat.workspace_bytes(D, lawcat.CALL_LAYER_PREFILL_FM)
    out = []
    for more in (0, 4 << 20):
        O, S, z = torch.empty_like(Q), torch.empty(1, 2, 64, 64, device="cuda"), torch.empty(1, 2, 64, device="cuda")
        ws = torch.empty(need + more, dtype=torch.uint8, device="cuda")
        lawcat.layer_prefill_fm(D, Q, K, V, G, wq, wk, H.dev(wf), None, None, None, None, O, None, S, z, None, None, ws)
        torch.cuda.synchronize()
        out.append((H.host(O), H.host(S), H.host(z)))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
