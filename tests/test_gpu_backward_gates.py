"""Gates that close within a chunk, and over whole segments: numbers of segments on both sides of where the boundary states'
combination changes from one launch to two, and every mixture of chunks that take their tokens together, in blocks and one by
one."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload, make_inputs, round_to_bf16

import helpers as H

pytestmark = pytest.mark.gpu


def _check(oracle, wl, gates, start, what):
    print("backward,", what, wl, "start state", start, flush=True)
    x = make_inputs(wl, seed=61, state=True)
    rnd = round_to_bf16 if wl.dtype == "bf16" else (lambda a: a)
    rng = np.random.default_rng(62)
    q, k = (rnd((np.abs(x[n]) + 0.05).astype(np.float32)) for n in ("Q", "K"))
    v, g = x["V"], rnd(gates(x["G"].copy(), rng).astype(np.float32))
    dO = rnd((rng.standard_normal(q.shape) * 0.5).astype(np.float32))
    S0, z0 = (x["S0"], np.abs(x["z0"]) + 0.5) if start else (None, None)
    den = oracle.gla_prefill(q, k, v, g, 1.0, 0.0, S0, z0)["den"].astype(np.float32)
    ref = oracle.gla_backward(q, k, v, g, dO, 1.0, 0.0, S0, z0)
    dt = H.tdtype(wl)
    desc = H.desc_for(wl)
    ins = [H.dev(a, dt) for a in (q, k, v, g)]
    outs = [torch.empty_like(t) for t in ins]
    dS0 = torch.empty(wl.B, wl.Hkv, wl.d, wl.d, device="cuda")
    dz0 = torch.empty(wl.B, wl.Hkv, wl.d, device="cuda")
    lawcat.gla_backward(desc, *ins, H.dev(den), H.dev(dO, dt), H.dev(S0), H.dev(z0), *outs, dS0, dz0,
                        lawcat.alloc_workspace(desc, lawcat.CALL_GLA_BACKWARD))
    torch.cuda.synchronize()
    for n, t in zip(("dq", "dk", "dv", "dg", "dS0", "dz0"), [*outs, dS0, dz0]):
        r = H.assert_close(H.host(t), ref[n], wl, f"{what}: {n}", 1 if wl.dtype == "bf16" and n in ("dq", "dk", "dv", "dg") else 0)
        print(f"  {n}: error / bar {r:.3f}", flush=True)


@pytest.mark.parametrize("start", [False, True])
@pytest.mark.parametrize("d,nseg,dtype", [(64, 2, "fp32"), (64, 8, "bf16"), (64, 9, "bf16"), (64, 8, "fp32"), (128, 5, "bf16"), (128, 6, "bf16"), (128, 6, "fp32")])
@pytest.mark.parametrize("closed", [0, "middle", -2])
def test_segment_with_every_gate_closed(oracle, d, nseg, dtype, closed, start):
    """Segments of 64 tokens: nothing of the state before a closed one is left after it, nothing of dS after it before it."""
    wl = Workload("closed", B=1, T=64 * nseg - 11, Hq=4, Hkv=2, d=d, dtype=dtype)
    i = nseg // 2 if closed == "middle" else closed % nseg

    def gates(g, rng):
        g[:, 64 * i:64 * (i + 1)] = -30.0
        return g

    _check(oracle, wl, gates, start, f"{nseg} segments, number {i} closed")


def _channel(level):
    def gates(g, rng):
        g[..., 3] = level
        return g
    return gates


def _tokens(g, rng):
    g[rng.random(g.shape[:3]) < 0.05] = -30.0
    return g


def _chunks(g, rng):
    """one channel at a level of its own in every 16 tokens"""
    level = rng.choice([0.0, -3.0, -8.0, -15.0, -30.0, -90.0], size=(g.shape[0], (g.shape[1] + 15) // 16, g.shape[2]))
    g[..., 7] = np.repeat(level, 16, axis=1)[:, :g.shape[1]]
    return g


GATES = {"channel -3": _channel(-3.0), "channel -8": _channel(-8.0), "channel -30": _channel(-30.0), "channel -100": _channel(-100.0),
         "tokens": _tokens, "chunks": _chunks, "wide": lambda g, rng: 12.0 * g}


@pytest.mark.parametrize("gates", GATES)
@pytest.mark.parametrize("Hq,Hkv,d,dtype", [(2, 2, 64, "fp32"), (8, 2, 64, "fp32"), (4, 1, 64, "bf16"), (6, 2, 64, "bf16"), (16, 2, 64, "bf16"),
                                            (4, 2, 128, "fp32"), (3, 1, 128, "fp32"), (8, 2, 128, "bf16"), (1, 1, 128, "bf16")])
def test_gates_that_close(oracle, Hq, Hkv, d, dtype, gates):
    """Every number of query heads a pass takes, one pass and two."""
    _check(oracle, Workload("gates", B=2, T=149, Hq=Hq, Hkv=Hkv, d=d, dtype=dtype), GATES[gates], True, gates)


@pytest.mark.parametrize("gates", ["tokens", "wide"])
@pytest.mark.parametrize("T,Hq", [(2048, 8), (2049, 8), (4096, 8), (4097, 8), (4097, 24)])
def test_workgroups_of_one_query_head(oracle, T, Hq, gates):
    """One query head per pass, segments of 64 tokens: 256 workgroups, 264, 512 and 520, on both sides of where the sweeps' forms change."""
    _check(oracle, Workload("heads", B=1, T=T, Hq=Hq, Hkv=8, d=64, dtype="bf16"), GATES[gates], True, gates)


@pytest.mark.parametrize("gates", ["tokens", "wide"])
@pytest.mark.parametrize("B", [64, 65])
@pytest.mark.parametrize("Hq", [16, 32])
def test_workgroups_of_several_query_heads(oracle, Hq, B, gates):
    """Two and four query heads per pass, one segment to each of 512 and 520 heads."""
    _check(oracle, Workload("heads", B=B, T=40, Hq=Hq, Hkv=8, d=64, dtype="bf16"), GATES[gates], True, gates)
