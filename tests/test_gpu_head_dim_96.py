"""The d = 96 instantiation of the sweep kernel and its pre-pass (192-byte LDS rows, six score steps, three column
blocks, twelve copies dealt to four waves), against the fp64 CPU oracle and against itself where bits must agree."""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 96
SCALE = float(np.float32(D ** -0.5))
F16, PAIRS = binding.FLAG_F16_ALWAYS, binding.FLAG_NO_F16


def inputs(seed, B, H, Lq, Lkv, gain=1.0):
    g = torch.Generator().manual_seed(seed)
    mk = lambda L, s: (s * torch.randn(B, H, L, D, generator=g)).to(torch.bfloat16)
    return [mk(Lq, gain), mk(Lkv, gain), mk(Lkv, 1.0), mk(Lq, 0.5), mk(Lkv, 0.5), mk(Lkv, 0.5)]


def run(t, flags, **kw):
    out = binding.attn_jvp_fwd_ex(*[x if x is None else x.to(DEV) for x in t], SCALE, kernel=binding.KERNEL_MFMA, flags=flags, **kw)
    torch.cuda.synchronize()
    return out


def check(got, t, label):
    """The interface's tolerances for bf16 inputs: 1e-2, 2e-2 of RMS and 1e-3."""
    ref = attn_jvp_ref(*[torch.zeros_like(t[1 if i in (4, 5) else 0]) if x is None else x for i, x in enumerate(t)], SCALE)
    for x, r, tol in zip(got, ref, (1e-2, 2e-2, 1e-3)):
        if x is None:
            continue
        x = x.float().cpu().double().numpy()
        err = np.abs(x - r).max() / (1.0 if tol == 1e-3 else np.sqrt((r ** 2).mean()))
        assert np.isfinite(x).all() and err <= tol, f"{label}: {err}"


@pytest.mark.parametrize("flags", [F16, PAIRS])
def test_every_key_length_up_to_five_blocks(flags):
    for Lkv in range(1, 162):
        t = inputs(Lkv, 1, 1, 40, Lkv)
        check(run(t, flags), t, f"Lkv={Lkv}")


@pytest.mark.parametrize("flags", [F16, PAIRS])
@pytest.mark.parametrize("Lq", [1, 31, 33, 127, 129, 256, 257])
def test_query_lengths_around_tile_edges(Lq, flags):
    t = inputs(1000 + Lq, 2, 3, Lq, 300)
    check(run(t, flags), t, f"Lq={Lq}")


@pytest.mark.parametrize("case", ["online", "null-kv", "null-kv-pairs", "no-tangents", "no-tangents-pairs", "no-tangents-online"])
def test_variants(case):
    gain = 8 ** 0.5 if "online" in case else 1.0
    t = inputs(len(case), 1, 2, 260, 1100, gain)
    if "null-kv" in case or "no-tangents" in case:
        t[4] = t[5] = None
    if "no-tangents" in case:
        t[3] = None
    flags = PAIRS if "pairs" in case else F16
    got = run(t, flags)
    check(got, t, case)
    tt = [None if x is None else x.transpose(1, 2).contiguous() for x in t]            # [B, L, H, d]: the same bits
    blhd = run(tt, flags, layout=binding.LAYOUT_BLHD)
    assert torch.equal(blhd[0].transpose(1, 2), got[0]) and torch.equal(blhd[2], got[2])
    if got[1] is not None:
        assert torch.equal(blhd[1].transpose(1, 2), got[1])


@pytest.mark.parametrize("tangents", ["all", "query", "none"])
def test_resident_workgroups_give_the_same_bits(tangents):
    """1152 tiles: more than two per resident workgroup in every variant (256 units, up to two workgroups each)."""
    t = inputs(7, 4, 24, 1500, 290)
    if tangents != "all":
        t[4] = t[5] = None
    if tangents == "none":
        t[3] = None
    a, b = run(t, F16), run(t, F16 | binding.FLAG_NO_RESIDENT)
    for x, y in zip(a, b):
        assert (x is None and y is None) or torch.equal(x, y)
    sub = [None if x is None else x[3:, 23:] for x in t]
    check([None if x is None else x[3:, 23:] for x in a], sub, "last head")
