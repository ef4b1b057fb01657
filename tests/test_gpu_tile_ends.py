"""First and last key blocks of the tile kernels against the fp64 CPU oracle: samples of fewer than four blocks, sweeps of one
block to a main loop and every length of tail, with a last block that is whole, one key short, or one key.

Tolerances: the ones of bf16 inputs, max |x - x_ref| / RMS <= 1e-2 (O), 2e-2 (tO), 1e-3 absolute (lse).
"""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("flags", [binding.FLAG_NO_F16, binding.FLAG_F16_ALWAYS], ids=["pairs", "f16"])
@pytest.mark.parametrize("names", [6, 4, 3])
@pytest.mark.parametrize("d", [64, 96, 128])
def test_key_blocks(d, names, flags):
    scale = float(np.float32(d ** -0.5))
    for blocks in (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13):
        for Lkv in (32 * blocks, 32 * blocks - 1, 32 * blocks - 31):
            g = torch.Generator().manual_seed(Lkv)
            t = [torch.randn(1, 2, L, d, generator=g).to(torch.bfloat16) for L in (130, Lkv, Lkv, 130, Lkv, Lkv)]
            t = t[:names] + [None] * (6 - names)
            got = binding.attn_jvp_fwd_ex(*[None if x is None else x.to(DEV) for x in t], scale, flags=flags)
            full = [torch.zeros_like(t[1 if i in (4, 5) else 0]) if x is None else x for i, x in enumerate(t)]
            ref = attn_jvp_ref(*full, scale)
            for x, r, name, tol in zip(got, ref, ("o", "to", "lse"), (1e-2, 2e-2, 1e-3)):
                if x is not None:
                    x = x.cpu().double().numpy()
                    # (one key without key tangents: tO is zero, a difference of terms of size |tS V|)
                    err = np.abs(x - r).max() / (1.0 if name == "lse" else max(np.sqrt((r ** 2).mean()), 0.1))
                    assert np.isfinite(x).all() and err <= tol, f"Lkv={Lkv} {name}: {err}"


@pytest.mark.parametrize("names", [6, 4, 3])
@pytest.mark.parametrize("d", [32, 64, 96, 128])
def test_key_blocks_fp32(d, names):
    """The fp32 tile kernel (a flag asks for it): 1e-5 of RMS up to 256 keys, 1.5e-5 sqrt(Lkv / 256) beyond."""
    scale = float(np.float32(d ** -0.5))
    for blocks in (1, 2, 3, 4, 5, 6, 9):
        for Lkv in (32 * blocks, 32 * blocks - 1, 32 * blocks - 31):
            g = torch.Generator().manual_seed(Lkv)
            t = [torch.randn(1, 2, L, d, generator=g) for L in (130, Lkv, Lkv, 130, Lkv, Lkv)]
            t = t[:names] + [None] * (6 - names)
            got = binding.attn_jvp_fwd_ex(*[None if x is None else x.to(DEV) for x in t], scale, flags=binding.FLAG_NO_F16)
            full = [torch.zeros_like(t[1 if i in (4, 5) else 0]) if x is None else x for i, x in enumerate(t)]
            ref = attn_jvp_ref(*full, scale)
            tol = 1e-5 * max(1.0, 1.5 * (Lkv / 256) ** 0.5 if Lkv > 256 else 1.0)
            for x, r, name in zip(got, ref, ("o", "to", "lse")):
                if x is not None:
                    x = x.cpu().double().numpy()
                    # (one key without key tangents: tO is zero, a difference of terms of size |tS V|)
                    err = np.abs(x - r).max() / (1.0 if name == "lse" else max(np.sqrt((r ** 2).mean()), 0.5))
                    assert np.isfinite(x).all() and err <= tol, f"Lkv={Lkv} {name}: {err}"
