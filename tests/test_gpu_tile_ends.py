"""First and last key blocks of the tile kernels against the fp64 CPU oracle: samples of fewer than four blocks, sweeps of one
block to a main loop and every length of tail, with a last block that is whole, one key short, or one key.

Tolerances: the ones of bf16 inputs, max |x - x_ref| / RMS <= 1e-2 (O), 2e-2 (tO), 1e-3 absolute (lse); fp32 inputs see below.
"""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(got, t, scale, tols):
    full = [torch.zeros_like(t[1 if i in (4, 5) else 0]) if x is None else x for i, x in enumerate(t)]
    ref = attn_jvp_ref(*full, scale)
    Lkv = t[1].shape[2]
    for x, r, name, tol in zip(got, ref, ("o", "to", "lse"), tols):
        if x is not None:
            x = x.cpu().double().numpy()
            # one key without key tangents: tO is zero, the difference of terms of size |tS V|, here about 1; a half of that
            size = 0.5 if name == "to" and Lkv == 1 and t[4] is None else np.sqrt((r ** 2).mean())
            err = np.abs(x - r).max() / (1.0 if name == "lse" else size)
            assert np.isfinite(x).all() and err <= tol, f"Lkv={Lkv} {name}: {err}"


def inputs(Lkv, d, names, dtype):
    g = torch.Generator().manual_seed(Lkv)
    t = [torch.randn(1, 2, L, d, generator=g).to(dtype) for L in (130, Lkv, Lkv, 130, Lkv, Lkv)]
    return t[:names] + [None] * (6 - names)


def run(t, scale, **kw):
    """Both layouts give the same bits, and outputs of the input dtype are those of 32 bits, rounded."""
    u = [None if x is None else x.to(DEV) for x in t]
    got = binding.attn_jvp_fwd_ex(*u, scale, **kw)
    far = [None if x is None else x.transpose(1, 2).contiguous() for x in u]
    for out_dtype in {torch.float32, t[0].dtype}:
        for layout, ins in ((binding.LAYOUT_BHLD, u), (binding.LAYOUT_BLHD, far)):
            other = binding.attn_jvp_fwd_ex(*ins, scale, out_dtype=out_dtype, layout=layout, **kw)
            for x, y in zip(got[:2], other[:2]):
                if x is not None:
                    assert torch.equal(x.to(out_dtype), y.transpose(1, 2) if layout == binding.LAYOUT_BLHD else y), (t[1].shape, out_dtype, layout)
            assert torch.equal(got[2], other[2]), (t[1].shape, out_dtype, layout)
    return got


@pytest.mark.parametrize("flags", [binding.FLAG_NO_F16, binding.FLAG_F16_ALWAYS], ids=["pairs", "f16"])
@pytest.mark.parametrize("names", [6, 4, 3])
@pytest.mark.parametrize("d", [64, 96, 128])
def test_key_blocks(d, names, flags):
    scale = float(np.float32(d ** -0.5))
    for blocks in (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13):
        for Lkv in (32 * blocks, 32 * blocks - 1, 32 * blocks - 31):
            t = inputs(Lkv, d, names, torch.bfloat16)
            check(run(t, scale, flags=flags), t, scale, (1e-2, 2e-2, 1e-3))


@pytest.mark.parametrize("names", [6, 4, 3])
@pytest.mark.parametrize("d", [32, 64, 96, 128])
def test_key_blocks_fp32(d, names):
    """The fp32 tile kernel (a flag asks for it): 1e-5 of RMS up to 256 keys, 1.5e-5 sqrt(Lkv / 256) beyond."""
    scale = float(np.float32(d ** -0.5))
    for blocks in (1, 2, 3, 4, 5, 6, 9):
        for Lkv in (32 * blocks, 32 * blocks - 1, 32 * blocks - 31):
            t = inputs(Lkv, d, names, torch.float32)
            tol = 1e-5 if Lkv <= 256 else 1.5e-5 * (Lkv / 256) ** 0.5
            check(run(t, scale, flags=binding.FLAG_NO_F16), t, scale, (tol, tol, tol))


@pytest.mark.parametrize("names", [6, 4, 3])
@pytest.mark.parametrize("d", [64, 96, 128])
def test_redone_tiles(d, names):
    """Scores of later keys far above the first block's: every tile is redone with the running maximum.  576 tiles, so that workgroups
    share a unit where they may; the heads repeat each other and must have the same bits."""
    scale = float(np.float32(d ** -0.5))
    g = torch.Generator().manual_seed(d)
    t = [torch.randn(1, 4, L, d, generator=g) for L in (700, 300, 300, 700, 300, 300)]
    t[1][:, :, 32:] *= 40.0
    t = [x.to(torch.bfloat16) for x in t][:names] + [None] * (6 - names)
    got = binding.attn_jvp_fwd_ex(*[None if x is None else x.repeat(1, 24, 1, 1).to(DEV) for x in t], scale, flags=binding.FLAG_NO_F16)
    few = [None if x is None else x[:, :4] for x in got]
    check(few, t, scale, (1e-2, 2e-2, 1e-3))
    for x, y in zip(got, few):
        assert x is None or (x.view(24, *y.shape[1:]) == y).all()


@pytest.mark.parametrize("names,Lkv", [(6, 70), (4, 70), (3, 70), (3, 300)])
@pytest.mark.parametrize("d", [64, 128])
def test_rows_almost_too_far_apart(d, names, Lkv):
    """[B,L,H,d] with just under 2^25 elements between rows, the most that the bf16 tile kernel takes: offsets inside a block of 32 rows
    come up to 2^31 bytes, in the tail (70 keys) and in the main loop (300).  The heads repeat each other, and each has the bits of few heads."""
    some, scale, Lq = 100, float(np.float32(d ** -0.5)), 3
    heads = ((1 << 25) // d - 1) // some * some
    g = torch.Generator().manual_seed(d)
    t = [torch.randn(1, some, L, d, generator=g).to(torch.bfloat16) for L in (Lq, Lkv, Lkv, Lq, Lkv, Lkv)][:names] + [None] * (6 - names)
    few = binding.attn_jvp_fwd_ex(*[None if x is None else x.to(DEV) for x in t], scale, flags=binding.FLAG_NO_F16, workspace=None)
    check([None if x is None else x[:, :4] for x in few], [None if x is None else x[:, :4] for x in t], scale, (1e-2, 2e-2, 1e-3))
    many = [None if x is None else x.to(DEV).transpose(1, 2).repeat(1, 1, heads // some, 1) for x in t]
    got = binding.attn_jvp_fwd_ex(*many, scale, flags=binding.FLAG_NO_F16, workspace=None, layout=binding.LAYOUT_BLHD)
    for x, want in zip(got[:2], few[:2]):
        if x is not None:
            assert (x.view(1, Lq, -1, some, d) == want.transpose(1, 2)[:, :, None]).all()
    assert (got[2].view(1, -1, some, Lq) == few[2][:, None]).all()
    del many, got
    torch.cuda.empty_cache()
