"""fp32 inputs whose magnitudes differ between keys, rows, columns or channels (d in {32, 64, 96, 128}, the matrix-core
kernel) against the fp64 CPU oracle.

The kernel forms its products from operands split into two scaled fp16 terms.  fp32 products know every element to
2^-24 of itself, so large values that carry no weight, and other rows' or columns' large values, must cost nothing:
errors are taken row by row and column by column, each over its own RMS, so that no large row or column hides a small one.

Tolerance: 1e-5 as everywhere up to 256 keys, plus 40 x 2^-24 x max|S| (the rounding of an fp32 score becomes a relative
error of the weights) with the maximum over the scores that carry weight, those within 30 nats of their row's largest.  A
row or column has fewer elements than the whole tensor, so its RMS comes out smaller than the tensor's now and then:
twice that.
"""
import numpy as np
import pytest
import torch

from oracle.attn_jvp_ref import attn_jvp_ref
from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NAMES = ("q", "k", "v", "tq", "tk", "tv")


def inputs(seed, Lq, Lkv, d, H=2):
    g = torch.Generator().manual_seed(seed)
    mk = lambda L: torch.randn(1, H, L, d, generator=g)
    return {n: mk(Lq if n in ("q", "tq") else Lkv) for n in NAMES}


def drop(t, keys, nats):
    """Channel 0 carries nothing but the mask: `keys` score `nats` below what they would."""
    d = t["q"].shape[-1]
    t["q"][..., 0] = 1.0
    t["tq"][..., 0] = 0.0
    t["k"][..., 0] = 0.0
    t["tk"][..., 0] = 0.0
    t["k"][:, :, keys, 0] = -nats * d ** 0.5


def sc(d):
    return float(np.float32(d ** -0.5))


def run(t, names=NAMES, kernel=binding.KERNEL_MFMA):
    d = t["q"].shape[-1]
    out = binding.attn_jvp_fwd_ex(*[t[n].to(DEV) if n in names else None for n in NAMES], sc(d), kernel=kernel)
    torch.cuda.synchronize()
    return [None if x is None else x.cpu().double().numpy() for x in out]


def errors(got, ref):
    """Largest error of a row over the row's RMS, and of a column over the column's (zero rows and columns must be zero)."""
    res = []
    for axis in (-1, -2):
        rms = np.sqrt((ref ** 2).mean(axis=axis))
        res.append(float((np.abs(got - ref).max(axis=axis) / np.maximum(rms, 1e-30)).max()))
    return res


def check(t, label, names=NAMES, rows=True, columns=True):
    d = t["q"].shape[-1]
    full = {n: t[n] if n in names else torch.zeros_like(t[n]) for n in NAMES}
    ref = attn_jvp_ref(*[full[n] for n in NAMES], sc(d))
    s = (t["q"].double() @ t["k"].double().transpose(-1, -2)) * sc(d)
    live = s > s.amax(-1, keepdim=True) - 30.0
    tol = 2 * (1e-5 + 40 * 2.0 ** -24 * float(s[live].abs().max()))
    got = run(t, names)
    report = []
    for x, r, name in zip(got, ref, ("o", "to")):
        if x is None:
            continue
        by_row, by_col = errors(x, r)
        report.append((name, by_row if rows else 0.0, by_col if columns else 0.0, np.isfinite(x).all()))
    lse = float(np.abs(got[2] - ref[2]).max())
    print(f"[{label} d={d}] " + " ".join(f"{n}: rows {a:.1e} columns {b:.1e}" for n, a, b, _ in report) + f" lse {lse:.1e} tol {tol:.1e}", flush=True)
    for name, by_row, by_col, finite in report:
        assert finite and by_row <= tol and by_col <= tol, f"{label} d={d} {name}: rows {by_row}, columns {by_col}, allowed {tol}"
    assert lse <= tol, f"{label} d={d} lse: {lse}"


DIMS = pytest.mark.parametrize("d", [32, 64, 96, 128])


@DIMS
@pytest.mark.parametrize("f", [1e3, 1e4, 1e6, 1e8, 1e12])
def test_large_values_of_keys_without_weight(f, d):
    """The first key block lies 80 nats below the rest, as a mask through K leaves it, and holds large V."""
    t = inputs(1, 150, 256, d)
    drop(t, slice(0, 32), 80.0)
    t["v"][:, :, :32] *= f
    check(t, f"v-first-block x {f:g}")
    if f == 1e6:
        check(t, "the same, query tangents only", names=("q", "k", "v", "tq"))
        check(t, "the same, no tangents", names=("q", "k", "v"))


@DIMS
@pytest.mark.parametrize("keys", [slice(0, 8), slice(100, 256, 8)])
def test_large_values_among_keys_with_weight(keys, d):
    t = inputs(2, 150, 256, d)
    drop(t, keys, 45.0)
    t["v"][:, :, keys] *= 1e7
    check(t, "v x 1e7 on some keys")


@DIMS
def test_dominant_keys_without_values(d):
    """Every row's largest weight, by 15 nats, goes to a key whose V and tV are zero.  By rows only: what is left to a row is
    e^-(its sink's score), a few e-folds more or less from row to row, so a column's error is that of its largest rows over an
    RMS that few rows make."""
    t = inputs(3, 150, 256, d)
    drop(t, slice(1, None), 15.0)
    t["v"][:, :, 0] = 0.0
    t["tv"][:, :, 0] = 0.0
    check(t, "zero-valued sink", columns=False)


@DIMS
def test_columns_of_different_magnitude(d):
    t = inputs(4, 150, 256, d)
    f = 10.0 ** (-9.0 * torch.arange(d) / (d - 1))
    t["v"] *= f
    t["tv"] *= f
    t["v"][..., 5] = 0.0
    t["tv"][..., 5] = 0.0
    check(t, "columns over nine decades, one of zeros", rows=False)


@DIMS
@pytest.mark.parametrize("names", [NAMES, ("q", "k", "v", "tq")], ids=["all", "query"])
@pytest.mark.parametrize("f", [1e-3, 1e-5, 1e-8])
def test_query_tangents_of_different_magnitude(f, names, d):
    """Half of the rows of every tile have query tangents f times the others'; without key tangents their tO is smaller by
    the same factor."""
    t = inputs(5, 150, 256, d)
    t["tq"][:, :, ::2] *= f
    if "tk" in names:              # ... and with them, if those are small as well
        t["tk"] *= f
        t["tv"] *= f
    check(t, f"tq rows x {f:g}", names=names, columns=False)


@DIMS
@pytest.mark.parametrize("f", [1e4, 1e8])
def test_large_tangents_of_keys_without_weight(f, d):
    t = inputs(6, 150, 256, d)
    drop(t, slice(0, 32), 80.0)
    t["tk"][:, :, :32, 1:] *= f
    check(t, f"tk-first-block x {f:g}")
    t = inputs(7, 150, 256, d)
    drop(t, slice(0, 32), 1e7 / d ** 0.5)              # a mask of -1e7 in K, seen by the query tangents too
    t["tq"][..., 0] = 1.0
    check(t, "mask of -1e7, tangents there")


@DIMS
def test_rows_without_tangents(d):
    """Zero query tangents in some rows and none elsewhere: their tO is exactly zero."""
    t = inputs(8, 150, 256, d)
    t["tq"][:, :, 100:] = 0.0
    check(t, "rows without tangents", names=("q", "k", "v", "tq"), columns=False)


@DIMS
@pytest.mark.parametrize("f", [1e4, 1e6, 1e9])
@pytest.mark.parametrize("which", ["q", "k", "tq", "tk", "some keys"])
def test_large_channel_that_the_other_side_leaves_out(which, f, d):
    """One channel of `which` is large and meets zeros: it adds nothing to any score."""
    t = inputs(9, 150, 256, d)
    for n in ("q", "k", "tq", "tk"):
        t[n][..., 1] = 0.0
    if which == "some keys":
        t["k"][:, :, 3::7, 1] = f
    else:
        t[which][..., 1] = f
    check(t, f"channel of {which} at {f:g}")


@DIMS
def test_mask_in_a_channel(d):
    """A channel masks every third key with -1e9; what the keys hold besides does not matter."""
    t = inputs(10, 150, 256, d)
    drop(t, slice(0, 256, 3), 1e9 / d ** 0.5)
    check(t, "mask of -1e9")


@DIMS
@pytest.mark.parametrize("Lkv", [33, 64, 95, 289])
def test_redone_tiles_at_block_edges(Lkv, d):
    """V of the first block is zero, so every tile is redone with fp32 products: one to ten key blocks, ragged and not, each set
    of tangents, both layouts.  (With 33 keys one alone has values: a row's tO is that key's V times the difference of two
    tangent scores, which comes near zero in some row, so rows are left out there.)"""
    t = inputs(11 + Lkv, 150, Lkv, d)
    t["v"][:, :, :32] = 0.0
    t["tv"][:, :, :32] = 0.0
    for names in (NAMES, ("q", "k", "v", "tq"), ("q", "k", "v")):
        check(t, f"redone, Lkv={Lkv}, {len(names)} tensors", names=names, rows=Lkv != 33)
        blhd = [t[n].transpose(1, 2).contiguous().to(DEV) if n in names else None for n in NAMES]
        got = binding.attn_jvp_fwd_ex(*blhd, sc(d), kernel=binding.KERNEL_MFMA, layout=binding.LAYOUT_BLHD)
        want = run(t, names)
        assert np.array_equal(got[0].transpose(1, 2).cpu().double().numpy(), want[0])
        assert np.array_equal(got[2].cpu().double().numpy(), want[2])
        if want[1] is not None:
            assert np.array_equal(got[1].transpose(1, 2).cpu().double().numpy(), want[1])


@DIMS
@pytest.mark.parametrize("names", [NAMES, ("q", "k", "v", "tq")], ids=["all", "query"])
@pytest.mark.parametrize("f", [1e-3, 1e-4])
def test_small_tangents_beside_large_ones_in_peaked_rows(f, names, d):
    """Logit std 8, where one key has most of many rows' weight and A + B cancels against r O: tO of the rows with small
    tangents together, error over result in the 2-norm.  fp32 products: 1.5e-6 to 3.4e-6; allowed three times that.  (Scaled
    for the other rows' tangents alone: 8e-6 at 1e-3, 7e-5 at 1e-4.)"""
    t = inputs(12, 384, 256, d)
    t["q"] *= 8 ** 0.5
    t["k"] *= 8 ** 0.5
    t["tq"][:, :, ::2] *= f
    t["tk"] *= f
    t["tv"] *= f
    full = {n: t[n] if n in names else torch.zeros_like(t[n]) for n in NAMES}
    ref = attn_jvp_ref(*[full[n] for n in NAMES], sc(d))[1][:, :, ::2]
    got = run(t, names)[1][:, :, ::2]
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(f"[small tangents x {f:g}, peaked, {len(names)} tensors, d={d}] {err:.1e}", flush=True)
    assert err <= 1e-5
