"""Segment start states on both sides of the change from folding (few segments) to the scan: every number of segments around it,
one head and many, with and without a start state, and with segments whose decay is exactly zero at either end."""
import numpy as np
import pytest

from paper_2509_18467_amd.inputs import Workload, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shut", [(), (0,), (1,), (0, 1)])
@pytest.mark.parametrize("d,B,Hkv,nseg", [
    # head dim 64 folds up to 9 segments with 2 heads, 11 with 8, 12 with 12 and more; 128 up to 4, 5, 7 with 24, and (groups below eight) 8 with 32, 9 with 40
    (64, 1, 2, 2), (64, 1, 2, 9), (64, 1, 2, 10), (64, 1, 8, 11), (64, 1, 8, 12), (64, 2, 8, 12), (64, 2, 8, 13),
    (128, 1, 2, 2), (128, 1, 2, 4), (128, 1, 2, 5), (128, 1, 8, 5), (128, 1, 8, 6), (128, 3, 8, 7), (128, 3, 8, 8), (128, 4, 8, 8), (128, 8, 8, 9), (128, 8, 8, 10)])
def test_start_states(oracle, d, B, Hkv, nseg, shut):
    wl = Workload("fold", B, 64 * nseg - 11, Hkv, Hkv, d, 4, "bf16")
    x = make_inputs(wl, seed=61, halo=True, state=not shut or shut == (1,))
    for s in shut:      # every channel closed over a whole segment: the first, or the one before the last
        at = 64 * (s * (nseg - 2))
        x["G"][:, at:at + 64] = -30.0
    print("segment start states", wl, shut, flush=True)
    got = H.run_layer_prefill(wl, x, segment=64, gate_scale=0.25)
    ref = oracle.layer_prefill(x["Q"], x["K"], x["V"], x["G"], x["wq"], x["wk"], 1, 0.25, 0.0, x.get("S0"), x.get("z0"),
                               x["q_halo"], x["k_halo"])
    for n in ("o", "den", "S", "z"):
        H.assert_close(got[n], ref[n], wl, n)


# groups whose output pass is one launch, of one, two or four query heads a workgroup, or (no multiple of 4, many heads) two, each of
# which folds: half as many segments
@pytest.mark.parametrize("shut", [(), (1,)])
@pytest.mark.parametrize("d,B,Hkv,group,nseg", [(64, 1, 2, 4, 6), (64, 1, 2, 4, 7), (64, 1, 1, 8, 3), (64, 1, 1, 8, 4), (64, 1, 1, 7, 2), (64, 4, 4, 16, 3), (64, 4, 4, 16, 4), (128, 1, 2, 2, 3), (128, 1, 2, 2, 4),
                                                (128, 4, 4, 8, 3), (128, 4, 4, 8, 4), (128, 4, 16, 4, 9), (128, 4, 16, 4, 10),
                                                (64, 2, 8, 6, 6), (64, 2, 8, 6, 7), (64, 4, 8, 7, 4), (64, 4, 8, 7, 5), (128, 4, 16, 6, 3), (128, 4, 16, 6, 4), (128, 4, 16, 6, 5),
                                                (128, 4, 8, 8, 7), (128, 4, 8, 8, 8)])
def test_start_states_of_several_output_launches(oracle, d, B, Hkv, group, nseg, shut):
    wl = Workload("fold", B, 64 * nseg - 11, Hkv * group, Hkv, d, 4, "bf16")
    x = make_inputs(wl, seed=62, halo=True, state=True)
    for s in shut:
        at = 64 * (s * (nseg - 2))
        x["G"][:, at:at + 64] = -30.0
    print("segment start states", wl, shut, flush=True)
    got = H.run_layer_prefill(wl, x, segment=64, gate_scale=0.25)
    ref = oracle.layer_prefill(x["Q"], x["K"], x["V"], x["G"], x["wq"], x["wk"], 1, 0.25, 0.0, x["S0"], x["z0"], x["q_halo"], x["k_halo"])
    for n in ("o", "den", "S", "z"):
        # closed gates leave an output of one product of a value with a weight that is rounded to bf16
        H.assert_close(got[n], ref[n], wl, n, 1 if shut and n == "o" else 0)
