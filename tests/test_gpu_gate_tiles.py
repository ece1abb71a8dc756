"""The gate projection around its tiles: 16 and 32 tokens, four and eight waves, input channels that leave some waves without a slab of
64 or with a last round that only some take, outputs that leave waves without a group of 128.  Against the oracle on the inputs as
stored."""
import numpy as np
import pytest

from paper_2509_18467_amd.inputs import Workload, make_gate_inputs

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 4096, 4097, 8191, 8192, 8193, 16353])
@pytest.mark.parametrize("dm,Hkv,d", [(128, 2, 64), (384, 9, 128), (1152, 8, 64)])
def test_gate_project_tiles(oracle, T, dm, Hkv, d):
    wl = Workload("gate", 1, T, Hkv, Hkv, d, 4, "bf16")
    gi = make_gate_inputs(wl, dm, 32, seed=54)
    print("gate_project tiles", wl, dm, flush=True)
    got = H.run_gate_project(wl, gi, dm, 32)
    ref = oracle.gate_project(gi["x"], gi["w1"], gi["w2"], gi.get("bias"), wl.Hkv)
    # the intermediate and the logits are rounded to bf16: half an ulp of the terms of the second product, and of the result
    h = np.asarray(gi["x"], dtype=np.float64) @ np.asarray(gi["w1"], dtype=np.float64).T
    terms = (np.abs(h) @ np.abs(np.asarray(gi["w2"], dtype=np.float64)).T).reshape(ref.shape)
    H.assert_close(got, ref, wl, "gate logits", roundings=1, terms=terms + np.abs(ref))


# tokens a workgroup: 12 with 7 in the last one, 14 with 3; 20 and 31 of eight waves, one left of 31; 17 and 28 with x of 1024 channels; 18 and
# 27 of four waves, two and three workgroups to a unit, 25 of four to a unit; 32 with x or outputs too narrow for that, and 16
@pytest.mark.parametrize("T,dm,Hkv", [(511, 2048, 2), (3335, 2048, 2), (5003, 2048, 2), (7906, 2048, 2), (4100, 1024, 2), (7000, 1024, 2),
                                      (8705, 1024, 2), (20480, 1024, 2), (24605, 2048, 16), (24605, 2048, 2), (5003, 256, 2), (8705, 256, 2),
                                      (3335, 1024, 2)])
def test_gate_project_shares(oracle, T, dm, Hkv):
    test_gate_project_tiles(oracle, T, dm, Hkv, 64)
