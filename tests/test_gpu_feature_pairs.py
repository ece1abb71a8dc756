"""The layer with the feature map, whose queries and keys are transformed in one launch: both head dimensions, groups that take four heads
a tile and one, every conv width, batches, lengths around a tile and several tiles a workgroup.  The transformed queries and keys bit
for bit as lawcat_conv1d_feature gives each, the rows kept exactly, the attention on them against the oracle."""
import numpy as np
import pytest

from paper_2509_18467_amd.inputs import Workload, make_feature_weights, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 3, 4, 8])
@pytest.mark.parametrize("B,T,W,halo,phi", [(1, 1, 4, True, 1), (2, 15, 4, False, 1), (3, 17, 4, True, 0), (1, 65, 3, True, 1), (2, 129, 2, True, 0), (1, 130, 1, False, 1),
                                            (2, 1500, 4, True, 1)])
def test_feature_pairs(oracle, d, group, B, T, W, halo, phi):
    wl = Workload("pairs", B, T, 2 * group, 2, d, W, "bf16")
    x = make_inputs(wl, seed=55, halo=halo and W > 1, state=halo)
    if phi == 0:       # no phi: features that keep the denominator from vanishing
        for n in ("Q", "K", "wq", "wk", "q_halo", "k_halo"):
            if n in x:
                x[n] = np.abs(x[n])
    wf = make_feature_weights(wl, seed=56)
    wf = wf if phi else np.abs(wf)
    print("feature pairs", wl, halo, phi, flush=True)
    got = H.run_layer_prefill(wl, x, feature_map=phi, wf=wf)
    for n, raw, w, h in (("q", "Q", "wq", "q_halo"), ("k", "K", "wk", "k_halo")):
        y, tail = H.run_conv_feature(wl, x[raw], x[w], wf, x.get(h), feature_map=phi)
        assert np.array_equal(got[n + "_dot"], y), n
        if W > 1:
            prev = np.zeros((B, W - 1, *x[raw].shape[2:])) if x.get(h) is None else x[h]
            assert np.array_equal(got[n + "_tail"], np.concatenate([prev, x[raw]], axis=1)[:, T:].astype(np.float64)), n
            assert np.array_equal(tail, got[n + "_tail"]), n
    f32 = np.float32
    ref = oracle.gla_prefill(got["q_dot"].astype(f32), got["k_dot"].astype(f32), x["V"], x["G"], 1.0, 0.0, x.get("S0"), x.get("z0"))
    for n in ("o", "den", "S", "z"):
        # (a few tokens are too few for an RMS: a half-ulp of the stored value beside it)
        H.assert_close(got[n], ref[n], wl, n, 1 if n == "o" else 0)
