"""lawcat_layer_prefill_static (the entry point that allocates nothing: its scratch is a static device array inside
the library) against lawcat_layer_prefill on the same inputs.  Both run the same kernels with the same segment
plan, so every output must agree bit for bit.  Two calls in a row share the one static buffer; the second one is
smaller, so it finds the first call's contents in the buffer."""
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import WORKLOADS, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)


def _both(wl, seed, quick=False):
    dt = H.tdtype(wl)
    x = make_inputs(wl, seed=seed, halo=True, state=True)
    desc = H.desc_for(wl, feature_map=1)
    ins = [H.dev(x[n], dt) for n in ("Q", "K", "V", "G", "wq", "wk")]
    S0, z0 = H.dev(x["S0"]), H.dev(x["z0"])
    qh, kh = H.dev(x["q_halo"], dt), H.dev(x["k_halo"], dt)

    def outputs():
        return [torch.full((wl.B, wl.T, wl.Hq, wl.d), float("nan"), dtype=dt, device="cuda"),
                torch.full((wl.B, wl.T, wl.Hq), float("nan"), device="cuda"),
                torch.full((wl.B, wl.Hkv, wl.d, wl.d), float("nan"), device="cuda"),
                torch.full((wl.B, wl.Hkv, wl.d), float("nan"), device="cuda"),
                torch.full((wl.B, wl.W - 1, wl.Hq, wl.d), float("nan"), dtype=dt, device="cuda"),
                torch.full((wl.B, wl.W - 1, wl.Hkv, wl.d), float("nan"), dtype=dt, device="cuda")]

    need = lawcat.workspace_bytes(desc, lawcat.CALL_LAYER_PREFILL)
    if quick:      # (only the least plan has to fit the limit)
        assert need > lawcat.STATIC_WORKSPACE_BYTES
    else:
        assert 0 < need <= lawcat.STATIC_WORKSPACE_BYTES, "the case must use the scratch buffer and fit it"
    ref = outputs()
    ws = lawcat.alloc_workspace(desc, lawcat.CALL_LAYER_PREFILL)
    lawcat.layer_prefill(desc, *ins, S0, z0, qh, kh, *ref, ws)
    got = outputs()
    lawcat.layer_prefill_static(desc, *ins, S0, z0, qh, kh, *got)
    torch.cuda.synchronize()
    for name, a, b in zip(("o", "den", "S", "z", "q_tail", "k_tail"), got, ref):
        assert not torch.isnan(a.float()).any(), f"{wl.name}: {name} holds unwritten elements"
        assert torch.equal(_bits(a), _bits(b)), f"{wl.name}: {name} differs from lawcat_layer_prefill"


def test_static_scratch_entry_point_matches_on_two_calls_in_a_row():
    print("no-alloc entry point: mistral7b shape T=9000, then llama1b shape T=3000", flush=True)
    _both(WORKLOADS["mistral7b_16k"].with_T(9000), seed=31)
    _both(WORKLOADS["llama1b_8k"].with_T(3000), seed=32)


def test_static_scratch_entry_point_matches_where_the_quickest_plan_needs_more_than_the_limit():
    print("no-alloc entry point: mistral7b shape T=18000", flush=True)
    _both(WORKLOADS["mistral7b_16k"].with_T(18000), seed=33, quick=True)
