"""What a token with an infinite operand or a zero denominator may spoil in the backward: its own gradients and those that
depend on it by the equations, nothing else.  Every gradient that does not depend on it is held to the bars of the ordinary
backward, against the oracle on inputs without it."""
import numpy as np
import pytest
import torch

from paper_2509_18467_amd import lawcat
from paper_2509_18467_amd.inputs import Workload, make_inputs, round_to_bf16

import helpers as H

pytestmark = pytest.mark.gpu

# one head per pass, two, four, and two passes; the token sits inside a 16-token chunk, in the first segment or the second
SHAPES = [(4, 2, 64, "fp32", 45, 21), (3, 1, 64, "bf16", 45, 21), (8, 2, 64, "bf16", 150, 83), (16, 2, 64, "bf16", 45, 21),
          (2, 2, 128, "fp32", 150, 83), (4, 1, 128, "bf16", 45, 21)]


def _inputs(Hq, Hkv, d, dtype, T, start):
    wl = Workload("finite", B=1, T=T, Hq=Hq, Hkv=Hkv, d=d, dtype=dtype)
    x = make_inputs(wl, seed=51, state=True)
    rnd = round_to_bf16 if dtype == "bf16" else (lambda a: a)
    q, k = (rnd((np.abs(x[n]) + 0.05).astype(np.float32)) for n in ("Q", "K"))
    dO = rnd((np.random.default_rng(52).standard_normal((1, T, Hq, d)) * 0.5).astype(np.float32))
    return wl, [q, k, x["V"], x["G"], dO], (x["S0"], np.abs(x["z0"]) + 0.5) if start else (None, None)


def _run(wl, q, k, v, g, dO, den, S0, z0):
    dt = H.tdtype(wl)
    desc = H.desc_for(wl)
    ins = [H.dev(a, dt) for a in (q, k, v, g)]
    outs = [torch.empty_like(t) for t in ins]
    lawcat.gla_backward(desc, *ins, H.dev(den), H.dev(dO, dt), H.dev(S0), H.dev(z0), *outs, None, None,
                        lawcat.alloc_workspace(desc, lawcat.CALL_GLA_BACKWARD))
    torch.cuda.synchronize()
    return dict(zip(("dq", "dk", "dv", "dg"), (H.host(t) for t in outs)))


def _check(wl, got, ref, what, **where):
    for n, sel in where.items():
        H.assert_close(got[n][sel], ref[n][sel], wl, f"{what}: {n}", 1 if wl.dtype == "bf16" else 0)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_padding_on_the_left(oracle, shape):
    """Tokens of zeros before the first one, no start state: their denominators are zero and their gradients NaN; those of
    the tokens after them are those of the sequence without the padding."""
    wl, x, _ = _inputs(*shape[:5], False)
    p = shape[-1]
    print("backward, padding", wl, p, flush=True)
    ref = oracle.gla_backward(*(a[:, p:] for a in x), 1.0, 0.0)
    for a in x[:3]:
        a[:, :p] = 0.0
    den = oracle.gla_prefill(*x[:4], 1.0, 0.0)["den"].astype(np.float32)
    assert not den[:, :p].any()
    got = _run(wl, *x, den, None, None)
    got = {n: a[:, p:] for n, a in got.items()}
    every = np.s_[:]
    _check(wl.with_T(wl.T - p), got, ref, "after the padding", dq=every, dk=every, dv=every, dg=every)


# closed: a channel that decays by 2^-10 a token, so that the chunks are cut into blocks whatever the values are
@pytest.mark.parametrize("closed", [False, True])
@pytest.mark.parametrize("which", ["q", "k", "v", "dO", "den"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_one_token_that_is_not_finite(oracle, shape, which, closed):
    Hq, Hkv, p = shape[0], shape[1], shape[-1]
    wl, x, start = _inputs(*shape[:5], True)
    if closed:
        x[3][:, :, :, 9] = -7.0
    print("backward, not finite:", which, wl, p, closed, flush=True)
    ref = oracle.gla_backward(*x, 1.0, 0.0, *start)
    den = oracle.gla_prefill(*x[:4], 1.0, 0.0, *start)["den"].astype(np.float32)
    if which == "den":
        den[0, p, Hq // Hkv - 1] = 0.0
    else:
        x["q k v g dO".split().index(which)][0, p, 0, 5] = np.inf
    got = _run(wl, *x, den, *start)
    before, after, others = np.s_[:, :p], np.s_[:, p + 1:], np.s_[:, :, 1:]
    if which in ("k", "v"):
        _check(wl, got, ref, "before", dq=before)
    else:
        _check(wl, got, ref, "after", dq=after, dk=after, dv=after, dg=after)
        _check(wl, got, ref, "before", dq=before)
    if Hkv > 1:
        _check(wl, got, ref, "the other kv heads", dq=np.s_[:, :, Hq // Hkv:], dk=others, dv=others, dg=others)


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[4] == 45], ids=str)
def test_a_key_too_large_to_be_divided_by_a_decay(oracle, shape):
    """A channel that decays by nearly 2^-64 over the chunk, and a key of 2^80 in it: the quotient would overflow."""
    wl, x, start = _inputs(*shape[:5], True)
    x[3][:, :, :, 5] = H.host(torch.tensor(-2.6875))
    p = 29
    print("backward, large key", wl, flush=True)
    before = np.s_[:, :p]
    ref = oracle.gla_backward(*x, 1.0, 0.0, *start)
    x[1][0, p, 0, 5] = 2.0 ** 80
    den = oracle.gla_prefill(*x[:4], 1.0, 0.0, *start)["den"].astype(np.float32)
    got = _run(wl, *x, den, *start)
    assert all(np.isfinite(a).all() for a in got.values())
    _check(wl, got, ref, "before the key", dq=before)


@pytest.mark.parametrize("which", ["q", "k", "v", "dO"])
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("level", [-2.6875, -3.5])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[4]], ids=str)
def test_tiny_and_huge_values_in_channels_that_nearly_close(oracle, shape, level, which, sign):
    """Chunks that decay by nearly 2^-60 and 2^-77, and operands scaled by a power of two: the gradients scale by powers of two as the
    equations say (eps = 0).  2^80 in fp32 storage; 2^64 in bf16 storage, whose products need 16 bits below an fp32 value."""
    power = sign * (80 if shape[3] == "fp32" else 64)
    wl, (q, k, v, g, dO), _ = _inputs(*shape[:5], False)
    g[:, :, 0] = level
    print("backward, scaled operand", wl, level, which, power, flush=True)
    den = oracle.gla_prefill(q, k, v, g, 1.0, 0.0)["den"].astype(np.float32)
    ref = _run(wl, q, k, v, g, dO, den, None, None)
    f = np.float32(2.0) ** np.float32(power)
    got = {"q": lambda: _run(wl, q * f, k, v, g, dO, den * f, None, None), "k": lambda: _run(wl, q, k * f, v, g, dO, den * f, None, None),
           "v": lambda: _run(wl, q, k, v * f, g, dO, den, None, None), "dO": lambda: _run(wl, q, k, v, g, dO * f, den, None, None)}[which]()
    scales = {"q": dict(dq=-1), "k": dict(dk=-1), "v": dict(dq=1, dk=1, dg=1), "dO": dict(dq=1, dk=1, dv=1, dg=1)}[which]
    # dg: a sum over the later tokens of differences of these, which nearly cancel; dq is such a difference itself, of terms
    # two to three times its size, and 2^-18 of those is 1e-5 of the RMS
    G = wl.Hq // wl.Hkv
    terms = np.abs(q * ref["dq"]).reshape(1, wl.T, wl.Hkv, G, wl.d).sum(axis=3) + np.abs(k * ref["dk"])
    terms = {"dg": np.cumsum(terms[:, ::-1], axis=1)[:, ::-1]}
    for n in ref:
        back = got[n] * 2.0 ** (-power * scales.get(n, 0))
        # powers of two change no rounding; a chunk walked in other blocks does: 64 fp32 ulps of the terms, and an ulp of
        # storage where they lie between two bf16 values
        lim = 1e-5 * H.rms(ref[n]) + H.FP32_REL * terms.get(n, 0.0) + (2 * H.BF16_HALF_ULP * np.abs(ref[n]) if wl.dtype == "bf16" else 0.0)
        ratio = np.abs(back - ref[n]) / lim
        print(f"  {n}: {ratio.max():.3f} of its bar", flush=True)
        assert ratio.max() <= 1.0, n


@pytest.mark.parametrize("which", ["q", "dO", "den"])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (4, 1), (8, 1)])
def test_not_finite_where_nothing_reaches_the_segments_start(oracle, which, Hq, Hkv):
    """Four query heads of 64 at a time: 50 tokens into the second segment the decay from its start, 2^-3.7 a token in every channel, is zero."""
    p = 114
    wl, x, start = _inputs(Hq, Hkv, 64, "bf16", 150, True)
    x[3][:] = -2.5
    print("backward, not finite far from the start:", which, wl, flush=True)
    ref = oracle.gla_backward(*x, 1.0, 0.0, *start)
    den = oracle.gla_prefill(*x[:4], 1.0, 0.0, *start)["den"].astype(np.float32)
    if which == "den":
        den[0, p, Hq // Hkv - 1] = 0.0
    else:
        x["q k v g dO".split().index(which)][0, p, 0, 5] = np.inf
    got = _run(wl, *x, den, *start)
    after = np.s_[:, p + 1:]
    _check(wl, got, ref, "after", dq=after, dk=after, dv=after, dg=after)
    _check(wl, got, ref, "before", dq=np.s_[:, :p])
