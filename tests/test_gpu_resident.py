"""Resident workgroups of the bf16 kernel where each walks through many tiles: the same bits as one workgroup per tile
(ATTN_JVP_FLAG_NO_RESIDENT).  Rows are checked against plain attention in fp64."""
import pytest
import torch

from paper_2510_08431_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def mk(seed, H, L, d, gain=1.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return (gain * torch.randn(1, H, L, d, generator=g, device=DEV)).to(torch.bfloat16)


def both_ways(args, scale, flags):
    res = binding.attn_jvp_fwd_ex(*args, scale, kernel=binding.KERNEL_MFMA, flags=flags)
    one = binding.attn_jvp_fwd_ex(*args, scale, kernel=binding.KERNEL_MFMA, flags=flags | binding.FLAG_NO_RESIDENT)
    torch.cuda.synchronize()
    for a, b in zip(res, one):
        assert (a is None and b is None) or torch.equal(a, b)
    return res


def handed_over(H, Lq):
    """Tiles that the last call's pair launch did: flags of 2 in the cached workspace, behind 32 bytes of statistics per head."""
    ws = binding._workspaces[(torch.device(DEV), torch.cuda.current_stream(DEV).cuda_stream)]
    off = (H * 32 + 255) // 256 * 256
    return int((ws[off:off + 4 * H * ((Lq + 127) // 128)].view(torch.int32) == 2).sum())


def check_rows(o, q, k, v, head, rows, scale):
    """O to 1e-2 of its RMS, as everywhere for bf16 inputs."""
    p = torch.softmax((q[0, head, rows].double() @ k[0, head].double().T) * scale, dim=-1)
    ref = p @ v[0, head].double()
    assert (o[0, head, rows].double() - ref).abs().max() <= 1e-2 * ref.pow(2).mean().sqrt()


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("case", ["f16", "pairs", "declined"])
def test_no_tangents_two_workgroups_per_unit(case, d):
    """Without tangents two workgroups share a compute unit at every head dimension, so the resident launch begins at four
    tiles per unit.  declined: logit std 6, every tile handed over to the pair kernel."""
    cus = torch.cuda.get_device_properties(DEV).multi_processor_count
    H, Lq, Lkv = -(-(4 * cus + 8) // 9), 1050, 300                # 9 tiles per head, the last ragged
    gain = 6.0 ** 0.5 if case == "declined" else 1.0
    q, k, v = mk(1, H, Lq, d, gain), mk(2, H, Lkv, d, gain), mk(3, H, Lkv, d)
    flags = {"f16": binding.FLAG_F16_ALWAYS, "pairs": binding.FLAG_NO_F16, "declined": 0}[case]
    o, to, _ = both_ways([q, k, v, None, None, None], d ** -0.5, flags)
    assert to is None
    if case != "pairs":
        assert handed_over(H, Lq) == (9 * H if case == "declined" else 0)
    for head in (0, H // 2, H - 1):
        check_rows(o, q, k, v, head, [0, 127, 128, 1023, 1024, 1049], d ** -0.5)


def test_hand_over_launch_with_more_than_64_tiles_per_workgroup():
    """A workgroup of a hand-over launch looks at the flags of 64 tiles at a time.  Here there are more than 64 per workgroup;
    the last head's tiles are declined (logit std 6), some of the second look among them (the launch deals each eighth of its
    tiles out in order, so that every eighth ends with some)."""
    cus = torch.cuda.get_device_properties(DEV).multi_processor_count
    H, d, Lkv = 4, 128, 256
    per_head = 64 * cus // H + 40                                 # tiles
    Lq = 128 * per_head - 5
    q, k, v = mk(4, H, Lq, d), mk(5, H, Lkv, d), mk(6, H, Lkv, d)
    q[:, H - 1] *= 6.0 ** 0.5
    k[:, H - 1] *= 6.0 ** 0.5
    tq, tk, tv = mk(7, H, Lq, d), mk(8, H, Lkv, d), mk(9, H, Lkv, d)
    o, _, _ = both_ways([q, k, v, tq, tk, tv], d ** -0.5, 0)
    assert handed_over(H, Lq) == per_head
    for head in (0, H - 2, H - 1):
        check_rows(o, q, k, v, head, [0, 128, Lq // 2, Lq - 128 * 30, Lq - 129, Lq - 1], d ** -0.5)
