"""Which workgroup of a packed batch takes which segment: one sequence, 64 (a wave's lanes) and more, lengths around multiples of the
segment and of a granule, by sequence, in order and by length.  Against the oracle, sequence by sequence."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload, make_inputs

import helpers as H

pytestmark = pytest.mark.gpu

RAGGED = (1, 63, 64, 65, 191, 192, 193, 384, 385, 577, 130, 320)


@pytest.mark.parametrize("d,Hkv,group,segment,lengths", [
    (64, 2, 2, 64, (130,)), (64, 2, 1, 64, RAGGED), (64, 2, 1, 64, (1,) * 64), (64, 1, 1, 128, (1, 129) * 33), (64, 1, 2, 64, (65, 1, 7) * 50),
    (64, 32, 4, 192, (500, 20, 200)),
    # a grid by sequences would not fit the chip, one by segments in order does
    (64, 2, 1, 64, (2000,) + (30,) * 20), (128, 2, 4, 64, (20, 900, 1, 63)),
    # nor that: by length
    (64, 16, 1, 192, RAGGED + (700, 700, 96)), (64, 12, 1, 192, (193, 40, 385, 192) * 16), (64, 8, 8, 192, RAGGED + (700, 700, 96)), (128, 16, 1, 192, RAGGED + (700, 96)),
    # more than 64 sequences: in order where that is the smaller grid
    (64, 4, 1, 64, (1,) * 70 + (1200,)), (128, 3, 2, 192, (20, 200) * 36)])
def test_packed_places(oracle, d, Hkv, group, segment, lengths):
    total, B = sum(lengths), len(lengths)
    wl = Workload("packed", 1, total, Hkv * group, Hkv, d, 4, "bf16")
    x = make_inputs(wl, seed=81)
    ext = make_inputs(Workload("packed", B, 1, Hkv * group, Hkv, d, 4, "bf16"), seed=82, halo=True, state=True)
    starts = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    print("packed places", wl, segment, B, flush=True)
    bf = torch.bfloat16
    D = lawcat.make_desc(B, max(lengths), wl.Hq, Hkv, d, feature_map=1, segment=segment, gate_scale=0.5)
    Q, K, V, G, wq, wk = (H.dev(x[n], bf) for n in ("Q", "K", "V", "G", "wq", "wk"))
    qh, kh, S0, z0 = H.dev(ext["q_halo"], bf), H.dev(ext["k_halo"], bf), H.dev(ext["S0"]), H.dev(ext["z0"])
    # (what no workgroup writes stays NaN)
    O, S, z, qt, kt = (torch.full_like(t, float("nan")) for t in (Q, S0, z0, qh, kh))
    den = torch.full((total, wl.Hq), float("nan"), dtype=torch.float32, device="cuda")
    need = lawcat.varlen_workspace_bytes(D, starts, True)
    ws = torch.full((max(need, 16) + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    lawcat.layer_prefill_varlen(D, starts, Q, K, V, G, wq, wk, S0, z0, qh, kh, O, den, S, z, qt, kt, ws[:max(need, 16)],
                                seq_start_dev=torch.from_numpy(starts).cuda())
    torch.cuda.synchronize()
    assert bool((ws[max(need, 16):] == 0x5A).all())
    o, dn, Sh, zh = H.host(O), H.host(den), H.host(S), H.host(z)
    for name, t in (("o", o), ("den", dn), ("S", Sh), ("z", zh), ("q_tail", H.host(qt)), ("k_tail", H.host(kt))):
        assert np.isfinite(t).all(), name
    for tail, raw, halo in ((qt, "Q", "q_halo"), (kt, "K", "k_halo")):
        tail = H.host(tail)
        for i, (a, b) in enumerate(zip(starts[:-1], starts[1:])):
            assert np.array_equal(tail[i], np.concatenate([ext[halo][i], x[raw][0, a:b]])[-3:].astype(np.float64)), i
    for i, (a, b) in enumerate(zip(starts[:-1], starts[1:])):
        if B > 20 and i % 7 and i != B - 1:      # (the oracle's time)
            continue
        ref = oracle.layer_prefill(x["Q"][:, a:b], x["K"][:, a:b], x["V"][:, a:b], x["G"][:, a:b], x["wq"], x["wk"], 1, 0.5, 0.0,
                                   ext["S0"][i:i + 1], ext["z0"][i:i + 1], ext["q_halo"][i:i + 1], ext["k_halo"][i:i + 1])
        got = {"o": o[0, a:b], "den": dn[a:b], "S": Sh[i], "z": zh[i]}
        for n in got:
            # (a few tokens are too few for an RMS: a half-ulp of the stored value beside it)
            H.assert_close(got[n][None], ref[n], wl, f"sequence {i} of {B - 1} {n}", roundings=1 if n == "o" else 0)
