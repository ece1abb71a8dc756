"""Output-pass workgroups that take four query heads of a group, two or one: group sizes around each, on both sides of the number of
segments at which the split changes, with a start state, conv caches and the smallest sequences; and calls in place, which are not
split."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu


# (walks = B x Hkv x segments of 64 tokens; a workgroup per query head up to 256 of them, per two heads up to 256, else per four)
@pytest.mark.parametrize("d,B,Hkv,group,T", [
    (64, 1, 2, 2, 1), (64, 1, 2, 3, 64), (64, 1, 1, 4, 65), (64, 2, 2, 6, 200), (64, 8, 8, 4, 64), (64, 8, 8, 4, 65), (64, 8, 16, 4, 60),
    (64, 16, 16, 4, 50), (64, 8, 8, 5, 64), (64, 8, 16, 3, 64), (64, 43, 2, 6, 65), (64, 16, 8, 8, 70), (128, 1, 2, 4, 1), (128, 1, 2, 3, 65), (128, 8, 8, 4, 64),
    (128, 8, 16, 4, 64), (128, 3, 8, 6, 250), (128, 4, 8, 8, 130)])
def test_groups(oracle, d, B, Hkv, group, T):
    wl = Workload("split", B, T, Hkv * group, Hkv, d, 4, "bf16")
    x = make_inputs(wl, seed=71, halo=True, state=True)
    print("head split", wl, flush=True)
    got = H.run_layer_prefill(wl, x, segment=64)
    ref = oracle.layer_prefill(x["Q"], x["K"], x["V"], x["G"], x["wq"], x["wk"], 1, 1.0, 0.0, x["S0"], x["z0"], x["q_halo"], x["k_halo"])
    for n in ("o", "den", "S", "z"):
        H.assert_close(got[n], ref[n], wl, n)
    for tail, raw, halo in (("q_tail", "Q", "q_halo"), ("k_tail", "K", "k_halo")):
        rows = np.concatenate([x[halo], x[raw]], axis=1)[:, -3:]
        assert np.array_equal(got[tail], rows.astype(np.float64))


@pytest.mark.parametrize("d", [64, 128])
def test_in_place(d):
    """One segment, the state's output over its input: as with buffers of their own, bit for bit in the state."""
    wl = Workload("split", 2, 60, 8, 2, d, 4, "bf16")
    x = make_inputs(wl, seed=72, halo=True, state=True)
    D = H.desc_for(wl, feature_map=1)
    Q, K, V, G, wq, wk, qh, kh = (H.dev(x[n], torch.bfloat16) for n in ("Q", "K", "V", "G", "wq", "wk", "q_halo", "k_halo"))
    out = []
    for inplace in (False, True):
        S0, z0, O = H.dev(x["S0"]), H.dev(x["z0"]), torch.empty_like(Q)
        S, z = (S0, z0) if inplace else (torch.empty_like(S0), torch.empty_like(z0))
        lawcat.layer_prefill(D, Q, K, V, G, wq, wk, S0, z0, qh, kh, O, None, S, z, None, None, None)
        torch.cuda.synchronize()
        out.append((H.host(O), H.host(S), H.host(z)))
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[0][2], out[1][2])
    # the outputs of another instantiation: the same products in the same order, up to how the compiler fuses them
    H.assert_close(out[1][0], out[0][0], wl, "o")
