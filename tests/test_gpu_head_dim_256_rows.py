"""Head dimension 256 with many query rows and few keys (one or two waves to 16 rows) against the fp64 CPU oracle; tolerance of
fp32 arithmetic as in test_gpu_keysplit.py."""
import pytest
import torch

from test_gpu_keysplit import DTYPES, check, inputs, run
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu


@DTYPES
@pytest.mark.parametrize("Lq,Lkv", [(250, 25), (256, 33), (241, 97), (193, 160)])
def test_edges_of_groups_and_blocks(dtype, Lq, Lkv):
    t = inputs(Lq + Lkv, 1, 128, Lq, Lkv, 256, dtype)
    for names in (6, 4, 3):
        u = t[:names] + [None] * (6 - names)
        check(run(u, 0.0625), u, 0.0625, f"{names} tensors")
    zero = t[:4] + [torch.zeros_like(t[4]), torch.zeros_like(t[5])]
    full, null = run(zero, 0.0625), run(t[:4] + [None, None], 0.0625)
    assert all(torch.equal(a, b) for a, b in zip(full, null))
    blhd = run([x.transpose(1, 2).contiguous() for x in t], 0.0625, layout=binding.LAYOUT_BLHD)
    want = run(t, 0.0625)
    assert torch.equal(blhd[0].transpose(1, 2), want[0]) and torch.equal(blhd[1].transpose(1, 2), want[1]) and torch.equal(blhd[2], want[2])


@DTYPES
def test_an_infinite_value_stays_in_its_column(dtype):
    """One group of a workgroup with an infinity: all its groups are redone with fp32 products, and only that column shows it."""
    t = inputs(4, 1, 128, 250, 60, 256, dtype)
    want = run(t, 0.0625)
    t[2][0, 5, 40, 3] = float("inf")
    o, to, lse = run(t, 0.0625)
    assert (o[0, 5, :, 3] == float("inf")).all()
    o[0, 5, :, 3], to[0, 5, :, 3] = want[0][0, 5, :, 3], want[1][0, 5, :, 3]
    for a, b in ((o, want[0]), (to, want[1])):
        assert (a - b).abs().max() <= 2e-5 * b.pow(2).mean().sqrt()
    assert (lse - want[2]).abs().max() <= 1e-5


@DTYPES
@pytest.mark.parametrize("Lkv", [1, 32])
def test_one_block_gives_the_bits_of_four_waves(dtype, Lkv):
    """One key block is one wave's either way: a call with few rows, which takes four waves to 16, has the same bits.  (One key has no
    entry in the test above: its to without key tangents is zero, the difference of equal terms of up to |tS V| = 20 here, each
    known to 2^-23, which no RMS of to measures: 2.4e-6 of 0.1 and more.)"""
    t = inputs(Lkv, 1, 128, 250, Lkv, 256, dtype)
    for names in (6, 4, 3):
        u = t[:names] + [None] * (6 - names)
        many, few = run(u, 0.0625), run([None if x is None else x[:, :2].contiguous() for x in u], 0.0625)
        assert all(x is None or torch.equal(x[:, :2], y) for x, y in zip(many, few))
