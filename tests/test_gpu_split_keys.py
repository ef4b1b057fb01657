"""Keys in parts (tile kernels on runs of the keys and a launch that merges them) against the fp64 CPU oracle.

Tolerances: fp32 inputs max |x - x_ref| / RMS(x_ref) <= 1e-5 up to 256 keys and 1.5e-5 sqrt(Lkv / 256) beyond, as the unsplit kernel.
bf16 inputs run as pairs, weights to 2^-17 of themselves: an o or to of a few effective keys is out by at most 2^-17 sum |w| |x|, with
|x| up to 5 times the RMS of a value and that up to 6 times the RMS of an o averaged over the keys here: 2.5e-4.
"""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

DEV = "cuda:0"
NAMES = ("q", "k", "v", "tq", "tk", "tv")
F32, BF16 = torch.float32, torch.bfloat16


def inputs(seed, B, H, Lq, Lkv, d, dtype, names=6):
    g = torch.Generator().manual_seed(seed)
    t = [torch.randn(B, H, Lq if n in ("q", "tq") else Lkv, d, generator=g).to(dtype) for n in NAMES]
    return t[:names] + [None] * (6 - names)


def run(t, scale, **kw):
    out = binding.attn_jvp_fwd_ex(*[None if x is None else x.to(DEV) for x in t], scale, **kw)
    torch.cuda.synchronize()
    return out


def check(got, t, scale, dtype):
    full = [torch.zeros_like(t[1 if i in (4, 5) else 0]) if x is None else x for i, x in enumerate(t)]
    ref = attn_jvp_ref(*full, scale)
    Lkv = t[1].shape[2]
    tol = 2.5e-4 if dtype == BF16 else 1e-5 if Lkv <= 256 else 1.5e-5 * (Lkv / 256) ** 0.5
    for x, r, name in zip(got, ref, ("o", "to", "lse")):
        if x is None:
            continue
        x = x.cpu().double().numpy()
        err = np.abs(x - r).max() / (1.0 if name == "lse" else np.sqrt((r ** 2).mean()))
        assert np.isfinite(x).all() and err <= tol, f"{name}: {err}"


# (the last column: keys, with the last part a whole run of blocks, a block and a key, or one key short of a block)
CASES = [(F32, 128, 1, 300, k) for k in (1024, 1025, 1055)] + [(F32, 64, 3, 129, 2001), (F32, 96, 2, 127, 1500), (F32, 32, 1, 130, 3000)] + \
        [(BF16, 128, 1, 300, k) for k in (2048, 2049, 2079)] + [(BF16, 64, 2, 257, 3000), (BF16, 96, 1, 128, 2500), (BF16, 32, 1, 200, 4001)]
IDS = ["%s-d%d-%dx%dx%d" % (("fp32" if c[0] == F32 else "bf16",) + c[1:]) for c in CASES]


def scratch_of(H, Lq, Lkv, d, dtype):
    lib = binding.load_library()
    return (lib.attn_jvp_workspace_bytes_fp32 if dtype == F32 else lib.attn_jvp_workspace_bytes)(1, H, Lq, Lkv, d)


def test_scratch_of_parts():
    """Host arithmetic: nothing for calls that fill the chip or have few keys, two states or more for the cases here, refused
    shapes and the ends of the integers included."""
    f32 = binding.load_library().attn_jvp_workspace_bytes_fp32
    assert f32(1, 2, 256, 256, 64) == 0 and f32(2, 16, 4096, 4096, 128) == 0 and f32(1, 1, 1000, 40, 128) == 0
    assert f32(1, 1, 1000, 1000, 256) == 0 and f32(0, 1, 1, 1, 64) == 0 and f32(1, 1, 300, 1024, -128) == 0
    assert f32(2**31 - 1, 2**31 - 1, 2**31 - 1, 2**31 - 1, 128) == 0
    for dtype, d, H, Lq, Lkv in CASES:
        if dtype == F32:
            assert scratch_of(H, Lq, Lkv, d, dtype) >= 2 * H * Lq * (8 * d + 16)


@pytest.mark.gpu
@pytest.mark.parametrize("names", [6, 4, 3])
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_parts_against_the_oracle(case, names):
    dtype, d, H, Lq, Lkv = case
    scale = float(np.float32(d ** -0.5))
    t = inputs(Lkv + names, 1, H, Lq, Lkv, d, dtype, names)
    got, whole = run(t, scale), run(t, scale, flags=binding.FLAG_NO_F16)
    check(got, t, scale, dtype)
    assert not torch.equal(got[0], whole[0])                  # (not on whole keys; in how many parts: test_numbers_of_parts)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [CASES[1], CASES[3], CASES[7], CASES[11]], ids=[IDS[1], IDS[3], IDS[7], IDS[11]])
def test_layouts_output_types_and_scratch(case):
    dtype, d, H, Lq, Lkv = case
    t = inputs(9, 2, H, Lq, Lkv, d, dtype)
    want = run(t, 0.1)
    blhd = run([x.transpose(1, 2).contiguous() for x in t], 0.1, layout=binding.LAYOUT_BLHD)
    assert torch.equal(blhd[0].transpose(1, 2), want[0]) and torch.equal(blhd[1].transpose(1, 2), want[1]) and torch.equal(blhd[2], want[2])
    for flags in (binding.FLAG_NO_RESIDENT, binding.FLAG_NO_LOCKSTEP):
        assert all(torch.equal(a, b) for a, b in zip(run(t, 0.1, flags=flags), want))
    low = run(t, 0.1, out_dtype=dtype)
    assert torch.equal(low[0], want[0].to(dtype)) and torch.equal(low[1], want[1].to(dtype)) and torch.equal(low[2], want[2])
    out = tuple(torch.empty_like(x) for x in want)
    dev = [x.to(DEV) for x in t]
    binding.attn_jvp_fwd_static(*dev, 0.1, out)
    torch.cuda.synchronize()
    own = {} if dtype == BF16 else {"workspace": None}      # (fp32: the entry point leaves its array alone)
    assert all(torch.equal(a, b) for a, b in zip(out, run(t, 0.1, **own)))
    need = scratch_of(2 * H, Lq, Lkv, d, dtype)
    guarded = torch.full((need + 512,), 0x5a, dtype=torch.uint8, device=DEV)
    exact = run(t, 0.1, workspace=guarded[:need])
    assert all(torch.equal(a, b) for a, b in zip(exact, want)) and (guarded[need:] == 0x5a).all()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.attn_jvp_fwd_static(*dev, 0.1, out)
    for rep in range(3):
        dev[0].mul_(0.9)
        eager = binding.attn_jvp_fwd_ex(*dev, 0.1, **own)
        for x in out:
            x.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, eager)), rep


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(F32, 128, 1, 300, 1024), (F32, 32, 1, 300, 3000), (BF16, 128, 4, 1100, 1100), (BF16, 64, 4, 1900, 1900)],
                         ids=["fp32-d128", "fp32-d32", "bf16-d128", "bf16-d64"])
def test_static_calls_that_need_no_scratch_leave_it_alone(case):
    """The library's array is one for all streams: only a call that has to use it does, so that the others may overlap."""
    dtype, d, H, Lq, Lkv = case
    t = [x.to(DEV) for x in inputs(10, 1, H, Lq, Lkv, d, dtype)]
    out = tuple(torch.empty(s, device=DEV) for s in ((1, H, Lq, d), (1, H, Lq, d), (1, H, Lq)))
    binding.attn_jvp_fwd_static(*t, 0.1, out)
    alone, parts = run(t, 0.1, workspace=None), run(t, 0.1)
    assert all(torch.equal(a, b) for a, b in zip(out, alone)) and not torch.equal(parts[0], alone[0])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d", [(F32, 128), (F32, 64), (BF16, 128), (BF16, 64)])
def test_a_part_without_weight(dtype, d):
    """Keys masked by an infinite element, whole parts of them: what counts is the softmax over the others."""
    Lkv, live = 3000, 700
    t = inputs(11, 1, 1, 140, Lkv, d, dtype, 3)
    t[0][..., 0] = 1.0
    t[1][:, :, live:, 0] = float("-inf")
    got = run(t, 0.1)
    rest = [t[0], t[1][:, :, :live].clone(), t[2][:, :, :live].clone(), None, None, None]
    check(got, rest, 0.1, dtype)
    t[1][:, :, 2900, 5] = float("nan")
    assert all(torch.isnan(x).all() for x in run(t, 0.1) if x is not None)


# the fewest rows and keys that go in each number of parts: (dtype, d, H, Lq, Lkv, tangents, parts)
COUNTS = [(BF16, 128, 8, 1300, 1033, 2, 2), (BF16, 128, 2, 3300, 1033, 2, 3), (BF16, 128, 2, 2100, 700, 2, 4), (BF16, 128, 2, 2100, 1033, 2, 5),
          (BF16, 128, 1, 300, 700, 2, 6), (BF16, 128, 1, 300, 1033, 2, 7), (BF16, 128, 1, 300, 1500, 2, 8), (BF16, 128, 8, 1300, 2077, 0, 2),
          (BF16, 64, 3, 2600, 1500, 0, 3), (BF16, 64, 2, 3300, 2077, 0, 4), (BF16, 64, 4, 1300, 2077, 2, 5), (BF16, 96, 8, 400, 2077, 2, 6),
          (BF16, 32, 8, 1100, 1500, 2, 3), (F32, 128, 6, 1300, 290, 2, 2), (F32, 128, 2, 2100, 290, 2, 3), (F32, 128, 2, 3300, 520, 2, 4),
          (F32, 128, 1, 300, 520, 2, 5), (F32, 64, 1, 300, 700, 2, 6), (F32, 96, 6, 1300, 700, 0, 3), (F32, 64, 2, 3300, 1033, 0, 4),
          (F32, 32, 3, 2100, 1500, 2, 5)]
COUNT_IDS = ["%s-d%d-%dx%dx%d-%d-%dparts" % (("fp32" if c[0] == F32 else "bf16",) + c[1:]) for c in COUNTS]


def route_of(case, tangents):
    dtype, d, H, Lq, Lkv = case[:5]
    return binding.attn_jvp_route(1, H, Lq, Lkv, d, 0.1, dtype, tangents=tangents)


def test_numbers_of_parts():
    """What the tests of this file run as (a call in parts is known without a GPU)."""
    assert {c[-1] for c in COUNTS if c[0] == BF16} == {2, 3, 4, 5, 6, 7, 8} and {c[-1] for c in COUNTS if c[0] == F32} >= {2, 3, 4, 5, 6}
    for case in COUNTS:
        assert route_of(case, case[5]) == ("f32-tiles" if case[0] == F32 else "bf16-pairs", case[6]), case
    for case in CASES:
        for tangents in (0, 1, 2):
            assert route_of(case, tangents)[1] >= 7, case


def check_rows(t, got, scale, dtype):
    """Every 29th row and the last one."""
    Lq = t[0].shape[2]
    rows = sorted(set(range(0, Lq, 29)) | {Lq - 1})
    cut = [x if x is None or i in (1, 2, 4, 5) else x[:, :, rows] for i, x in enumerate(t)]
    check([x if x is None else x[:, :, rows] for x in got], cut, scale, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("case", COUNTS, ids=COUNT_IDS)
def test_each_number_of_parts_against_the_oracle(case):
    dtype, d, H, Lq, Lkv, tangents, parts = case
    assert route_of(case, tangents)[1] == parts
    scale = float(np.float32(d ** -0.5))
    t = inputs(Lkv + parts, 1, H, Lq, Lkv, d, dtype, (3, 4, 6)[tangents])
    check_rows(t, run(t, scale), scale, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [128, 96, 64])
def test_workgroups_that_walk_through_tiles_of_several_parts(d):
    """Two tiles per compute unit and more, so that a workgroup goes on to another tile, of another part."""
    case = (BF16, d, 4, 3300, 20000)
    assert route_of(case, 2) == ("bf16-pairs", 7)                  # 104 query tiles, 728 workgroups' worth
    scale = float(np.float32(d ** -0.5))
    t = inputs(d, 1, 4, 3300, 20000, d, BF16)
    got = run(t, scale)
    assert all(torch.equal(a, b) for a, b in zip(got, run(t, scale, flags=binding.FLAG_NO_RESIDENT)))
    check_rows(t, got, scale, BF16)
