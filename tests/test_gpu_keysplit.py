"""The kernel that deals the keys of 16 query rows to the waves of a workgroup (calls with few rows, and head dimension 256)
against the fp64 CPU oracle, and the rule that takes calls to it.

Tolerance: max |x - x_ref| / RMS(x_ref) <= 1e-5 up to 256 keys and 1.5e-5 sqrt(Lkv / 256) beyond, the one of fp32 arithmetic
everywhere, for bf16 inputs too: their products are exact and their weights carry 24 bits.
"""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NAMES = ("q", "k", "v", "tq", "tk", "tv")
DTYPES = pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
LAUNCH_FLAGS = (binding.FLAG_NO_RESIDENT, binding.FLAG_NO_LOCKSTEP, binding.FLAG_NO_RESIDENT | binding.FLAG_NO_LOCKSTEP)      # results are identical
DIMS = pytest.mark.parametrize("d", [32, 64, 96, 128, 256])


def inputs(seed, B, H, Lq, Lkv, d, dtype):
    g = torch.Generator().manual_seed(seed)
    return [torch.randn(B, H, Lq if n in ("q", "tq") else Lkv, d, generator=g).to(dtype) for n in NAMES]


def run(t, scale, **kw):
    out = binding.attn_jvp_fwd_ex(*[None if x is None else x.to(DEV) for x in t], scale, **kw)
    torch.cuda.synchronize()
    return out


def check(got, t, scale, label):
    full = [torch.zeros_like(t[1 if i in (4, 5) else 0]) if x is None else x for i, x in enumerate(t)]
    ref = attn_jvp_ref(*full, scale)
    Lkv = t[1].shape[2]
    tol = 1e-5 if Lkv <= 256 else 1.5e-5 * (Lkv / 256) ** 0.5
    for x, r, name in zip(got, ref, ("o", "to", "lse")):
        if x is None:
            continue
        x = x.cpu().double().numpy()
        # (one key without key tangents: tO is zero, the difference of terms of size |tS V|, here about 1, each known to 2^-23 of it:
        # with 0.1 as the least RMS those 2^-22 are 2.4e-6)
        err = np.abs(x - r).max() / (1.0 if name == "lse" else max(np.sqrt((r ** 2).mean()), 0.1))
        assert np.isfinite(x).all() and err <= tol, f"{label} {name}: {err}"


@DTYPES
@DIMS
def test_key_and_query_lengths_around_the_edges(d, dtype):
    """Blocks of 32 keys dealt to four waves (waves without a block, with one, with several), tiles of 16 rows."""
    scale = float(np.float32(d ** -0.5))
    for Lq, Lkv in ((1, 1), (15, 31), (16, 32), (17, 33), (31, 64), (33, 97), (5, 127), (16, 128), (20, 129), (18, 161), (40, 300)):
        t = inputs(Lq + Lkv, 1, 2, Lq, Lkv, d, dtype)
        for names in (6, 4, 3):
            u = t[:names] + [None] * (6 - names)
            got = run(u, scale)
            check(got, u, scale, f"d={d} Lq={Lq} Lkv={Lkv} {names} tensors")
        blhd = run([x.transpose(1, 2).contiguous() for x in t], scale, layout=binding.LAYOUT_BLHD)
        full = run(t, scale)
        assert torch.equal(blhd[0].transpose(1, 2), full[0]) and torch.equal(blhd[1].transpose(1, 2), full[1]) and torch.equal(blhd[2], full[2])


@DTYPES
@DIMS
def test_absent_tangents_give_the_bits_of_zero_ones(d, dtype):
    t = inputs(3, 2, 2, 50, 200, d, dtype)
    zero = t[:4] + [torch.zeros_like(t[4]), torch.zeros_like(t[5])]
    full, null, plain = run(zero, 0.1), run(t[:4] + [None, None], 0.1), run(t[:3] + [None] * 3, 0.1)
    assert all(torch.equal(a, b) for a, b in zip(full, null))
    assert plain[1] is None and torch.equal(plain[0], full[0]) and torch.equal(plain[2], full[2])


@DTYPES
@DIMS
def test_infinities_and_nan_stay_in_their_columns(d, dtype):
    """One element of V: infinite, the column's o is that infinity (its weights are positive); NaN, NaN; the rest is right."""
    t = inputs(4, 1, 1, 20, 150, d, dtype)
    scale = float(np.float32(d ** -0.5))
    want = run(t, scale)
    for bad in (float("inf"), float("-inf"), float("nan")):
        u = [x.clone() for x in t]
        u[2][0, 0, 70, 3] = bad
        o, to, lse = run(u, scale)
        col = o[..., 3]
        assert (torch.isnan(col) if bad != bad else col == bad).all()
        rest = [i for i in range(d) if i != 3]
        for a, b in ((o, want[0]), (to, want[1])):
            assert (a[..., rest] - b[..., rest]).abs().max() <= 2e-5 * b.pow(2).mean().sqrt()
        assert (lse - want[2]).abs().max() <= 1e-5


@pytest.mark.parametrize("d,dtype,kernel", [(64, torch.float32, binding.KERNEL_MFMA), (128, torch.bfloat16, binding.KERNEL_AUTO),
                                            (32, torch.bfloat16, binding.KERNEL_AUTO), (96, torch.float32, binding.KERNEL_AUTO)])
def test_route_by_rows_and_flags(d, dtype, kernel):
    """Few rows come here (fp32 accuracy shows it for bf16 inputs), a flag asks for the tile kernel, many rows go there."""
    scale = float(np.float32(d ** -0.5))
    t = inputs(5, 1, 2, 200, 300, d, dtype)
    few, tile = run(t, scale, kernel=kernel), run(t, scale, kernel=kernel, flags=binding.FLAG_NO_F16)
    check(few, t, scale, "few rows")
    assert not torch.equal(few[0], tile[0])
    for flags in LAUNCH_FLAGS:
        assert all(torch.equal(x, y) for x, y in zip(few, run(t, scale, kernel=kernel, flags=flags)))
    many = inputs(6, 1, 16, 5 * 16 * 17, 40, d, dtype)             # 85 groups of 16 rows a head, 1360 in all
    a, b = run(many, scale, kernel=kernel), run(many, scale, kernel=kernel, flags=binding.FLAG_NO_F16)
    assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_static_scratch_and_graph_with_more_rows_than_this_kernel_takes():
    """The fp16 value path of the tile kernel through the entry point that brings its own scratch, captured in a HIP graph: every
    replay the bits of an eager call."""
    B, H, Lq, Lkv, d = 1, 12, 730, 2100, 128
    t = [x.to(DEV) for x in inputs(7, B, H, Lq, Lkv, d, torch.bfloat16)]
    out = (torch.empty(B, H, Lq, d, device=DEV), torch.empty(B, H, Lq, d, device=DEV), torch.empty(B, H, Lq, device=DEV))
    binding.attn_jvp_fwd_static(*t, 0.1, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.attn_jvp_fwd_static(*t, 0.1, out)
    for rep in range(3):
        t[0].mul_(0.9)
        eager = binding.attn_jvp_fwd_ex(*t, 0.1)
        for x in out:
            x.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, eager)), rep


@DTYPES
@DIMS
def test_sums_of_large_values_stay_finite(d, dtype):
    """Equal weights on values up to 3e38: o is their mean, however many there are; the same for tV, whose overflow alone must not move o."""
    kw = {} if d == 96 and dtype == torch.bfloat16 else {"workspace": None}      # (which needs one to be taken at all)
    for Lkv in (100, 300, 1000) if kw else (100, 300):
        t = inputs(8, 1, 1, 20, Lkv, d, dtype)
        t[0].zero_()
        t[3].mul_(2.0 ** -10)
        for which in ((2, 5), (5,)):
            u = list(t)
            for i in which:
                u[i] = ((t[i].float().abs().clamp(max=3.0) + 0.1) * 2.0 ** 126).to(dtype)      # 8.5e37 * (0.1 .. 3.1)
            got = run(u, 0.1, **kw)
            ref = attn_jvp_ref(*u, 0.1)
            for x, r, name in zip(got[:2], ref, ("o", "to")):
                x = x.cpu().double().numpy()
                assert np.isfinite(x).all() and np.abs(x - r).max() <= 2e-5 * np.sqrt((r ** 2).mean()), f"{name} {which} Lkv={Lkv}"
            plain = run(u[:3] + [None] * 3, 0.1, **kw)
            assert torch.equal(plain[0], got[0]) and torch.equal(plain[2], got[2])


@DTYPES
@DIMS
def test_rows_without_a_finite_score(d, dtype):
    """lse is the logarithm of an empty sum, whichever kernel has the call; o has no value."""
    own = {} if d == 96 and dtype == torch.bfloat16 else {"workspace": None}      # (which needs one to be taken at all)
    for Lkv in (1, 100, 1500):
        t = [x.to(dtype) for x in (torch.ones(1, 1, 20, d), torch.randn(1, 1, Lkv, d), torch.randn(1, 1, Lkv, d))] + [None] * 3
        t[1][..., 0] = float("-inf")
        for kw in ({}, own) + (({"flags": binding.FLAG_NO_F16},) if d in (64, 128) else ()):
            o, _, lse = run(t, 0.1, **kw)
            assert torch.isnan(o).all() and (lse == float("-inf")).all(), (Lkv, kw)
        t[1][0, 0, Lkv - 1] = float("nan")
        assert torch.isnan(run(t, 0.1, **own)[2]).all()


@pytest.mark.parametrize("d,dtype,names", [(64, torch.float32, 6), (128, torch.bfloat16, 4), (32, torch.bfloat16, 4), (64, torch.float32, 3)])
def test_either_side_of_one_workgroup_per_compute_unit(d, dtype, names):
    """Up to there a workgroup has a unit's registers to itself, beyond two share them: the same bits for the same rows."""
    cus = torch.cuda.get_device_properties(DEV).multi_processor_count
    scale = float(np.float32(d ** -0.5))
    t = inputs(9, 1, 1, 16 * cus + 5, 130, d, dtype)
    t = t[:names] + [None] * (6 - names)
    head = lambda n: [x if x is None else x[:, :, :n].contiguous() if i in (0, 3) else x for i, x in enumerate(t)]
    two, one = run(t, scale, workspace=None), run(head(16 * cus), scale, workspace=None)
    for a, b in zip(two, one):
        assert a is None or torch.equal(a[:, :, :16 * cus], b)
    check(run(head(40), scale, workspace=None), head(40), scale, "one")


@pytest.mark.parametrize("names", [6, 4, 3])
@pytest.mark.parametrize("d,heads,Lkv", [(32, 1048600, 33), (64, 524300, 70), (96, 349600, 40), (128, 600000, 40)])
def test_rows_far_apart(d, heads, Lkv, names):
    """[B,L,H,d] with 2^25 elements between rows and more: a key block's rows reach beyond 2^31 and 2^32 bytes.  The heads repeat each
    other, and each has the bits that it has in a call with few heads."""
    some, scale, Lq = 100, float(np.float32(d ** -0.5)), 3
    t = inputs(11, 1, some, Lq, Lkv, d, torch.bfloat16)
    t = t[:names] + [None] * (6 - names)
    few = run(t, scale)
    assert binding.attn_jvp_route(1, some, Lq, Lkv, d, scale, tangents={6: 2, 4: 1, 3: 0}[names])[0] == "keysplit"
    check([None if x is None else x[:, :4] for x in few], [None if x is None else x[:, :4] for x in t], scale, "few heads")
    many = [None if x is None else x.to(DEV).transpose(1, 2).repeat(1, 1, heads // some, 1) for x in t]
    # (head dimensions 32 and 96 are taken with a workspace only, which this kernel leaves alone)
    ws = None if d in (64, 128) else torch.empty(binding.attn_jvp_workspace_bytes(1, heads, Lq, Lkv, d), dtype=torch.uint8, device=DEV)
    for flags in (0, binding.FLAG_NO_F16):
        got = run(many, scale, workspace=ws, layout=binding.LAYOUT_BLHD, flags=flags)
        for x, want in zip(got[:2], few[:2]):
            if x is not None:
                assert (x.view(1, Lq, -1, some, d) == want.transpose(1, 2)[:, :, None]).all()
        assert (got[2].view(1, -1, some, Lq) == few[2][:, None]).all()
    del many, got, ws
    torch.cuda.empty_cache()
