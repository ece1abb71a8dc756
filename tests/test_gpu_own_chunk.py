"""Which wave of the output pass takes which of a granule's four chunks (head dim 64: all of one; 128: scores and denominators of one):
lengths around chunks and granules, every number of query heads a workgroup takes (few sequences one, in place all of a group up to four,
many sequences by their number), chunks whose decay is referred to their middle, alone and beside ordinary ones, gate logits without
bound."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu

LENGTHS = (1, 15, 16, 17, 49, 63, 64, 65, 81, 129, 191)


def _in_place(wl, x, segment):
    """S_out, z_out over S0, z0: a workgroup takes as many query heads of a group as it can."""
    desc = H.desc_for(wl, feature_map=1, segment=segment)
    Q, K, V, G, wq, wk, qh, kh = (H.dev(x[n], torch.bfloat16) for n in ("Q", "K", "V", "G", "wq", "wk", "q_halo", "k_halo"))
    S, z, O, den = H.dev(x["S0"]), H.dev(x["z0"]), torch.empty_like(Q), torch.empty(*Q.shape[:-1], device="cuda")
    lawcat.layer_prefill(desc, Q, K, V, G, wq, wk, S, z, qh, kh, O, den, S, z, None, None, lawcat.alloc_workspace(desc, lawcat.CALL_LAYER_PREFILL))
    torch.cuda.synchronize()
    return {"o": H.host(O), "den": H.host(den), "S": H.host(S), "z": H.host(z)}


def _shut(x, shut):
    for c in shut:      # three tokens of the chunk in every other channel: far past the decay that the chunk's start can refer to
        x["G"][:, 16 * c + 5:16 * c + 8, :, ::2] = -40.0


@pytest.mark.parametrize("shut", [(), (2,), (0, 5)])
@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("T", LENGTHS)
def test_chunks(oracle, T, group, shut):
    wl = Workload("own", 1, T, 2 * group, 2, 64, 4, "bf16")
    x = make_inputs(wl, seed=81, halo=True, state=True)
    _shut(x, shut)
    print("own chunk", wl, shut, flush=True)
    ref = oracle.layer_prefill(x["Q"], x["K"], x["V"], x["G"], x["wq"], x["wk"], 1, 1.0, 0.0, x["S0"], x["z0"], x["q_halo"], x["k_halo"])
    # one walk of the whole sequence and segments of a granule, by workgroups of one query head and, in place, of all the group's
    for segment, run in ((192, H.run_layer_prefill), (64, H.run_layer_prefill), (192, _in_place), (64, _in_place)):
        got = run(wl, x, segment=segment)
        for n in ("o", "den", "S", "z"):
            H.assert_close(got[n], ref[n], wl, n)


@pytest.mark.parametrize("shut", [(), (1, 3)])
@pytest.mark.parametrize("d,B,group", [(64, 64, 2), (64, 65, 2), (64, 64, 4), (64, 65, 4), (128, 64, 2), (128, 65, 2), (128, 64, 4), (128, 65, 4)])
def test_many_heads(oracle, d, B, group, shut):
    """128 and 130 walks: of two query heads a workgroup takes one and two, of four two and four."""
    wl = Workload("own", B, 70, 2 * group, 2, d, 4, "bf16")
    x = make_inputs(wl, seed=85, halo=True, state=True)
    _shut(x, shut)
    print("many heads", wl, shut, flush=True)
    got = H.run_layer_prefill(wl, x, segment=128)
    ref = oracle.layer_prefill(x["Q"], x["K"], x["V"], x["G"], x["wq"], x["wk"], 1, 1.0, 0.0, x["S0"], x["z0"], x["q_halo"], x["k_halo"])
    for n in ("o", "den", "S", "z"):
        H.assert_close(got[n], ref[n], wl, n)


@pytest.mark.parametrize("shut", [(), (1, 3)])
@pytest.mark.parametrize("group", [2, 4])
def test_without_conv_many_heads(oracle, group, shut):
    """More workgroups than compute units, so that one takes two or four query heads; queries and keys as they are."""
    wl = Workload("own", 35, 70, 8 * group, 8, 64, 4, "bf16")
    x = make_inputs(wl, seed=82, state=True)
    _shut(x, shut)
    q, k = np.abs(x["Q"]), np.abs(x["K"])
    got = H.run_gla_prefill(wl, q, k, x["V"], x["G"], x["S0"], x["z0"])
    ref = oracle.gla_prefill(q, k, x["V"], x["G"], 1.0, 0.0, x["S0"], x["z0"])
    for n in ("o", "den", "S", "z"):
        H.assert_close(got[n], ref[n], wl, n)


@pytest.mark.parametrize("shut", [(), (0, 5)])
@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("T", (1, 16, 17, 49, 64, 81, 191))
def test_chunks_of_128_channels(oracle, T, group, shut):
    wl = Workload("own", 1, T, 2 * group, 2, 128, 4, "bf16")
    x = make_inputs(wl, seed=83, halo=True, state=True)
    _shut(x, shut)
    print("own chunk", wl, shut, flush=True)
    ref = oracle.layer_prefill(x["Q"], x["K"], x["V"], x["G"], x["wq"], x["wk"], 1, 1.0, 0.0, x["S0"], x["z0"], x["q_halo"], x["k_halo"])
    for segment, run in ((192, H.run_layer_prefill), (64, H.run_layer_prefill), (192, _in_place), (64, _in_place)):
        got = run(wl, x, segment=segment)
        for n in ("o", "den", "S", "z"):
            H.assert_close(got[n], ref[n], wl, n)


@pytest.mark.parametrize("d", [64, 128])
def test_unbounded_logits(oracle, d):
    """Logits of -200 and of -infinity close a channel as -30 does: e^200 and infinity both end at the floor of the decay."""
    wl = Workload("own", 1, 200, 8, 2, d, 4, "bf16")
    x = make_inputs(wl, seed=84, halo=True, state=True)
    out = []
    for low in (-30.0, -200.0, -np.inf):
        x["G"][:, 40:150:7, :, ::3] = low
        out.append(H.run_layer_prefill(wl, x, segment=64))
    for got in out[1:]:
        for n in ("o", "den", "S", "z"):
            assert np.array_equal(got[n], out[0][n])
