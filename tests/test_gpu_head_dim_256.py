"""The fp32 matrix-core kernel for head dimension 256 (what KERNEL_AUTO and KERNEL_FP32 run there) against the fp64 CPU
oracle.  Tolerance: max |x - x_ref| / RMS(x_ref) <= 1e-5 up to 256 keys, the one for fp32 arithmetic everywhere."""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 256
SCALE = 1 / 16


def inputs(seed, B, H, Lq, Lkv, dtype, gain=1.0):
    g = torch.Generator().manual_seed(seed)
    mk = lambda L, s: (s * torch.randn(B, H, L, D, generator=g)).to(dtype)
    return [mk(Lq, gain), mk(Lkv, gain), mk(Lkv, 1.0), mk(Lq, 1.0), mk(Lkv, 1.0), mk(Lkv, 1.0)]


def run(t, scale=SCALE, **kw):
    out = binding.attn_jvp_fwd_ex(*[None if x is None else x.to(DEV) for x in t], scale, **kw)
    torch.cuda.synchronize()
    return out


def check(got, t, label, scale=SCALE, tol=1e-5):
    ref = attn_jvp_ref(*t, scale)
    for x, r, name in zip(got, ref, ("o", "to", "lse")):
        x = x.cpu().double().numpy()
        err = np.abs(x - r).max() / (1.0 if name == "lse" else max(np.sqrt((r ** 2).mean()), 1e-3))
        assert np.isfinite(x).all() and err <= tol, f"{label} {name}: {err}"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_every_key_length_up_to_three_blocks(dtype):
    for Lkv in range(1, 50):
        t = inputs(Lkv, 1, 1, 20, Lkv, dtype)
        check(run(t), t, f"Lkv={Lkv}")


@pytest.mark.parametrize("Lq", [1, 15, 17, 63, 64, 65, 130])
def test_query_lengths_around_tile_edges(Lq):
    t = inputs(100 + Lq, 2, 3, Lq, 70, torch.float32)
    check(run(t), t, f"Lq={Lq}")


@pytest.mark.parametrize("scale", [0.0, -0.07])
def test_non_positive_scale(scale):
    t = inputs(9, 1, 2, 40, 37, torch.bfloat16)
    scale = float(np.float32(scale))
    check(run(t, scale), t, f"scale={scale}", scale)


def test_peaked_rows_move_the_reference():
    """Logit std 64: a block's maximum often exceeds the reference by more than its 32 nats.  An fp32 score of size |S| is
    known to a few 2^-24 |S|, which the exponential turns into a relative error: 40 x 2^-24 x max|S| on top."""
    t = inputs(11, 1, 2, 70, 200, torch.float32, gain=8.0)
    s_max = float((t[0].double() @ t[1].double().transpose(-1, -2)).abs().max()) * SCALE
    check(run(t), t, "peaked", tol=1e-5 + 40 * 2.0 ** -24 * s_max)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_absent_tangents_and_layout_give_the_same_bits(dtype):
    t = inputs(12, 2, 3, 70, 45, dtype)
    zero = [x if i < 4 else torch.zeros_like(x) for i, x in enumerate(t)]
    full, null = run(zero), run(zero[:4] + [None, None])
    assert all(torch.equal(a, b) for a, b in zip(full, null))
    plain = run(t[:3] + [None] * 3)
    assert plain[1] is None and torch.equal(plain[0], full[0]) and torch.equal(plain[2], full[2])
    got = run(t)
    tt = [x.transpose(1, 2).contiguous() for x in t]
    blhd = run(tt, layout=binding.LAYOUT_BLHD)
    assert torch.equal(blhd[0].transpose(1, 2), got[0]) and torch.equal(blhd[1].transpose(1, 2), got[1]) and torch.equal(blhd[2], got[2])
    rounded = run(t, out_dtype=dtype)
    assert torch.equal(rounded[0], got[0].to(dtype)) and torch.equal(rounded[1], got[1].to(dtype))


def test_keys_at_minus_infinity_weigh_nothing():
    """More than a key block of them in front, and one at the end."""
    t = inputs(13, 1, 1, 20, 60, torch.float32)
    t[0] = t[0].abs() + 0.1
    dead = list(range(20)) + [59]
    t[1][:, :, dead] = float("-inf")
    o, _, lse = run(t[:3] + [None] * 3)
    live = [i for i in range(60) if i not in dead]
    cut = [x if i in (0, 3) else x[:, :, live] for i, x in enumerate(t)]
    ref = attn_jvp_ref(*cut, SCALE)
    assert np.abs(o.cpu().double().numpy() - ref[0]).max() <= 1e-5 * np.sqrt((ref[0] ** 2).mean())
    assert np.abs(lse.cpu().double().numpy() - ref[2]).max() <= 1e-5


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_values_near_the_end_of_the_range_under_rising_scores(dtype):
    """Scores rise by 25 nats along the keys (the reference follows, the weights stay at most 1): V, tV of 1e36 must not
    overflow, as they do not in O and tO.  Inputs scaled down by the same factor give the same numbers, up to the rounding
    of that factor."""
    t = inputs(14, 1, 2, 40, 100, dtype, gain=0.25)
    t[0][..., 0] = 4.0
    t[1][..., 0] = torch.arange(100).to(dtype) * (1 / SCALE) / 4 * 0.25
    for x in (t[3], t[4]):
        x.mul_(2.0 ** -6)
    big = [x * 2.0 ** 119 if i in (2, 5) else x for i, x in enumerate(t)]       # (an exact factor)
    small, large = run(t), run(big)
    check(small, t, "rising scores", tol=1e-5 + 40 * 2.0 ** -24 * 30)
    for a, b in zip(small[:2], large[:2]):
        assert torch.isfinite(b).all() and torch.equal(b, a * 2.0 ** 119)
    assert torch.equal(small[2], large[2])
