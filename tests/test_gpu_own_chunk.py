"""Head dim 64, where a wave of the output pass takes one of a granule's four chunks: lengths around chunks and granules, every number of
query heads a workgroup takes, chunks whose decay is referred to their middle, alone and beside ordinary ones."""
import numpy as np
import pytest

from paper_2509_18467_amd.inputs import Workload, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu

LENGTHS = (1, 15, 16, 17, 49, 63, 64, 65, 81, 129, 191)


@pytest.mark.parametrize("shut", [(), (2,), (0, 5)])
@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("T", LENGTHS)
def test_chunks(oracle, T, group, shut):
    wl = Workload("own", 1, T, 2 * group, 2, 64, 4, "bf16")
    x = make_inputs(wl, seed=81, halo=True, state=True)
    for c in shut:      # three tokens of the chunk in every other channel: far past the decay that the chunk's start can refer to
        x["G"][:, 16 * c + 5:16 * c + 8, :, ::2] = -40.0
    print("own chunk", wl, shut, flush=True)
    ref = oracle.layer_prefill(x["Q"], x["K"], x["V"], x["G"], x["wq"], x["wk"], 1, 1.0, 0.0, x["S0"], x["z0"], x["q_halo"], x["k_halo"])
    # one walk of the whole sequence, segments of a granule, and (most: the heads a workgroup takes go by the workgroups there are)
    for segment in (192, 64):
        got = H.run_layer_prefill(wl, x, segment=segment)
        for n in ("o", "den", "S", "z"):
            H.assert_close(got[n], ref[n], wl, n)


@pytest.mark.parametrize("group", [2, 4])
def test_without_conv_many_heads(oracle, group):
    """More workgroups than compute units, so that one takes two or four query heads; queries and keys as they are."""
    wl = Workload("own", 35, 70, 8 * group, 8, 64, 4, "bf16")
    x = make_inputs(wl, seed=82, state=True)
    q, k = np.abs(x["Q"]), np.abs(x["K"])
    got = H.run_gla_prefill(wl, q, k, x["V"], x["G"], x["S0"], x["z0"])
    ref = oracle.gla_prefill(q, k, x["V"], x["G"], 1.0, 0.0, x["S0"], x["z0"])
    for n in ("o", "den", "S", "z"):
        H.assert_close(got[n], ref[n], wl, n)
