"""Numbers so small that the bf16 terms of the key-split kernel do not hold them, against the oracle in 64 bits.

Tolerance: 1e-5 of the RMS of a row and of a column, the one of fp32 arithmetic; twice that because a row or column has fewer elements
than the whole tensor.  Inputs are at least 1e-36, so that their products with weights of ordinary size stay normal numbers.
"""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NAMES = ("q", "k", "v", "tq", "tk", "tv")
TOL = 2e-5
F32, BF16 = torch.float32, torch.bfloat16
DIMS = pytest.mark.parametrize("d", [32, 64, 96, 128, 256])


def inputs(seed, d, dtype=F32, Lq=40, Lkv=200):
    g = torch.Generator().manual_seed(seed)
    return {n: torch.randn(1, 2, Lq if n in ("q", "tq") else Lkv, d, generator=g).to(dtype) for n in NAMES}


def run(t, names=NAMES, **kw):
    d = t["q"].shape[-1]
    out = binding.attn_jvp_fwd_ex(*[t[n].to(DEV) if n in names else None for n in NAMES], float(np.float32(d ** -0.5)), **kw)
    torch.cuda.synchronize()
    return out


def check(t, label, columns=True):
    d = t["q"].shape[-1]
    ref = attn_jvp_ref(*[t[n] for n in NAMES], float(np.float32(d ** -0.5)))
    got = run(t)
    worst = []
    for x, r in zip(got[:2], ref):
        err = np.abs(x.cpu().double().numpy() - r)
        worst += [float((err / np.sqrt((r ** 2).mean(axis=axis, keepdims=True))).max()) for axis in ((-1, -2) if columns else (-1,))]
    lse = float(np.abs(got[2].cpu().double().numpy() - ref[2]).max())
    print(f"[{label} d={d}] o, to by rows and columns " + " ".join(f"{e:.1e}" for e in worst) + f" lse {lse:.1e}", flush=True)
    assert max(worst) <= TOL and lse <= 1e-5, label


@DIMS
@pytest.mark.parametrize("f", [1e-24, 1e-30, 1e-34, 1e-36])
def test_values(f, d):
    t = inputs(1, d)
    t["v"] *= f
    t["tv"] *= f
    check(t, f"v, tv x {f:g}")
    t = inputs(2, d)
    t["v"][..., 5] *= f
    t["tv"][..., 5] *= f
    check(t, f"a column of v, tv x {f:g}")


@DIMS
@pytest.mark.parametrize("f", [1e-24, 1e-30, 1e-34, 1e-36])
def test_tangents(f, d):
    t = inputs(3, d)
    for n in ("tq", "tk", "tv"):
        t[n] *= f
    check(t, f"tangents x {f:g}")
    t["v"] /= f
    t["tv"] /= f
    check(t, f"tq, tk x {f:g}, v over it")
    t = inputs(4, d)
    t["tq"][:, :, ::2] = 0.0
    t["tk"] *= f
    t["tv"] *= f
    t["tq"][:, :, 1::2] *= f
    check(t, f"tk, tv and half of the rows of tq x {f:g}, the other half without")


@DIMS
@pytest.mark.parametrize("f", [1e-12, 1e-24, 1e-34, 1e-36])
@pytest.mark.parametrize("small", ["q", "k"])
def test_one_side_of_the_scores_against_the_other(small, f, d):
    t = inputs(5, d)
    large = "k" if small == "q" else "q"
    for n in (small, "t" + small):
        t[n] *= f
    for n in (large, "t" + large):
        t[n] /= f
    check(t, f"{small} x {f:g}, {large} over it")


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("f", [2.0 ** -100, 2.0 ** -115])
def test_bf16_inputs(f, d):
    """Exact in one term each; the products of weights and tangent scores are not."""
    t = inputs(6, d, BF16)
    for n in ("tq", "tk"):
        t[n] *= f
    t["v"] /= f
    check(t, f"bf16, tq, tk x {f:g}, v over it")
    t = inputs(7, d, BF16)
    t["v"] *= f
    t["tv"] *= f
    check(t, f"bf16, v, tv x {f:g}")


@DIMS
def test_o_and_lse_have_the_same_bits_whatever_the_tangents(d):
    """Also where a tile is done again because of its tangents, small or infinite."""
    t = inputs(8, d)
    want = run(t, NAMES[:3])
    for n in ("tq", "tk", "tv"):
        t[n] *= 1e-34
    for u in (t, {**t, "tv": t["tv"].clone()}):
        if u is not t:
            u["tv"][0, 0, 7, 3] = float("inf")
        got = run(u)
        assert torch.equal(got[0], want[0]) and torch.equal(got[2], want[2])
    assert torch.isinf(got[1][0, 0, :, 3]).all()
    t["v"] *= 1e-34
    got, want = run(t), run(t, NAMES[:3])
    assert torch.equal(got[0], want[0]) and torch.equal(got[2], want[2])
