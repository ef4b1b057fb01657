"""The native way of an ordinary call (csrc/fast_call.cpp) against the Python one, which takes every call that names a stream."""
import os
import subprocess
import sys
import threading

import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2510_08431_amd import binding

DEV = "cuda:0"
BF16, F32 = torch.bfloat16, torch.float32


class Sub(torch.Tensor):
    pass


def native(t, scale=0.1, out_dtype=F32, kernel=0, flags=0, layout=0, with_workspace=True):
    binding.load_library()
    return binding._fast.attn(*t, scale, out_dtype, kernel, flags, layout, with_workspace)


def test_what_is_not_a_plain_gpu_call_is_left_to_python():
    binding.load_library()
    x = torch.zeros(1, 1, 8, 64)
    assert native([x] * 6) is None and native([x] * 5 + [None]) is None and native([1, 2, 3, 4, 5, 6]) is None
    assert binding._fast.rmsnorm(x, x, torch.ones(64), 1e-6) is None and binding._fast.rmsnorm(x, x, None, 1e-6) is None
    assert binding._fast.attn(x) is None
    with pytest.raises(ValueError, match="must live on the GPU"):
        binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1)
    with pytest.raises(ValueError, match="must live on the GPU"):
        binding.attn_jvp_rmsnorm_fwd(x, x, torch.ones(64), 1e-6)


def inputs(dtype, B=2, H=3, Lq=37, Lkv=70, d=64):
    g = torch.Generator().manual_seed(1)
    return [torch.randn(B, H, L, d, generator=g).to(dtype).to(DEV) for L in (Lq, Lkv, Lkv, Lq, Lkv, Lkv)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [F32, BF16], ids=["fp32", "bf16"])
def test_same_results_as_the_python_way(dtype):
    stream = torch.cuda.current_stream()
    shapes = ({}, {"Lq": 1, "Lkv": 1}, {"Lq": 1, "H": 1, "Lkv": 3001, "d": 128}, {"Lq": 900, "Lkv": 2100, "d": 128}, {"d": 256}, {"d": 32, "Lkv": 2500})
    for kw in shapes:
        t = inputs(dtype, **kw)
        for names in (6, 4, 3):
            u = t[:names] + [None] * (6 - names)
            for opts in ({}, {"out_dtype": dtype}, {"layout": binding.LAYOUT_BLHD}, {"workspace": None}):
                a = [x if x is None or "layout" not in opts else x.transpose(1, 2).contiguous() for x in u]
                assert native(a, out_dtype=opts.get("out_dtype", F32), layout=opts.get("layout", 0)) is not None
                got, want = binding.attn_jvp_fwd_ex(*a, 0.1, **opts), binding.attn_jvp_fwd_ex(*a, 0.1, stream=stream, **opts)
                for x, y in zip(got, want):
                    assert (x is None and y is None) or (torch.equal(x, y) and x.dtype == y.dtype and x.stride() == y.stride()), (kw, names, opts)
        if dtype == BF16 and t[0].shape[-1] in (64, 128):
            assert all(torch.equal(x, y) for x, y in zip(binding.attn_jvp_fwd(*t, 0.1), binding.attn_jvp_fwd_ex(*t, 0.1, stream=stream, workspace=None)))
    x, w = inputs(dtype)[0], torch.rand(64, device=DEV)
    assert all(torch.equal(a, b) for a, b in zip(binding.attn_jvp_rmsnorm_fwd(x, 2 * x, w, 1e-6), binding.attn_jvp_rmsnorm_fwd(x, 2 * x, w, 1e-6, stream=stream)))


@pytest.mark.gpu
def test_refused_calls_and_watched_calls():
    t = inputs(BF16)
    for i, bad in ((1, t[1][..., :32]), (1, t[1].transpose(2, 3)), (2, t[2].float()), (0, t[0][0]), (5, None), (3, None)):
        u = list(t)
        u[i] = bad
        with pytest.raises((ValueError, AttributeError)):
            binding.attn_jvp_fwd_ex(*u, 0.1)
    with pytest.raises(binding.AttnJvpError):
        binding.attn_jvp_fwd_ex(*[x[..., :48].contiguous() for x in t], 0.1)
    with pytest.raises(binding.AttnJvpError):
        binding.attn_jvp_rmsnorm_fwd(t[0][..., :48].contiguous(), t[0][..., :48].contiguous(), torch.ones(48, device=DEV), 1e-6)
    want = binding.attn_jvp_fwd_ex(*t, 0.1)
    sub = [t[0].as_subclass(Sub)] + t[1:]
    assert native(sub) is None and torch.equal(binding.attn_jvp_fwd_ex(*sub, 0.1)[0], want[0])

    class Watch(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            Watch.seen += 1
            return func(*args, **(kwargs or {}))

    with Watch():
        got = binding.attn_jvp_fwd_ex(*t, 0.1)
    assert Watch.seen >= 3 and torch.equal(got[0], want[0])
    with pytest.raises(RuntimeError):
        torch.vmap(lambda q: binding.attn_jvp_fwd_ex(q, *t[1:], 0.1)[0])(torch.stack([t[0], t[0]]))


@pytest.mark.gpu
@pytest.mark.filterwarnings("ignore:Named tensors")
def test_outputs_take_over_what_the_python_way_takes_over():
    """Dimension names of q and x; in inference mode the outputs are inference tensors."""
    stream = torch.cuda.current_stream()
    q, w = inputs(BF16, Lkv=37)[0], torch.ones(64, device=DEV)
    for named in (False, True):
        x = q.rename("B", "H", "L", "D") if named else q
        calls = (lambda **kw: binding.attn_jvp_fwd_ex(*[x] * 6, 0.1, **kw), lambda **kw: binding.attn_jvp_rmsnorm_fwd(x, x, w, 1e-6, **kw))
        for call in calls:
            for mode in (torch.no_grad, torch.inference_mode):
                with mode():
                    got, want = call(), call(stream=stream)
                for a, b in zip(got, want):
                    assert a.names == b.names and a.is_inference() == b.is_inference() == (mode is torch.inference_mode)
                    assert torch.equal(a.rename(None), b.rename(None))
        assert (got[0].names == x.names) and (got[0].names[-1] == "D") == named


@pytest.mark.gpu
def test_streams_and_threads():
    """Every thread its own stream: each call on its thread's current stream with that stream's workspace."""
    t = inputs(BF16, Lq=300, Lkv=2100, d=128, H=1)
    want = binding.attn_jvp_fwd_ex(*t, 0.1)
    torch.cuda.synchronize()
    wrong = []

    def work():
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(20):
                got = binding.attn_jvp_fwd_ex(*t, 0.1)
                stream.synchronize()
                if not all(torch.equal(a, b) for a, b in zip(got, want)):
                    wrong.append(1)
        if (torch.device(DEV), stream.cuda_stream) not in binding._workspaces:
            wrong.append(2)

    threads = [threading.Thread(target=work) for _ in range(4)]
    [x.start() for x in threads]
    [x.join() for x in threads]
    assert not wrong


CHILD = """
import sys, warnings
sys.path.insert(0, sys.argv[1])
import torch
from paper_2510_08431_amd import binding
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    assert binding.load_library().attn_jvp_version() > 0
assert binding.__file__.startswith(sys.argv[1])
x = torch.zeros(1, 1, 8, 64)
for call in (lambda: binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1), lambda: binding.attn_jvp_rmsnorm_fwd(x, x, torch.ones(64), 1e-6),
             lambda: binding.attn_jvp_fwd(*[x.bfloat16()] * 6, 0.1)):
    try:
        call()
        raise SystemExit("accepted CPU tensors")
    except ValueError as e:
        assert "must live on the GPU" in str(e)
print([str(w.message) for w in seen if "_fast_call" in str(w.message)])
"""


@pytest.mark.parametrize("module,content,reason", [(None, None, "cannot import name '_fast_call'"), ("_fast_call.so", b"not a library", "file too short"),
                                                   ("_fast_call.py", b"torch_version = '1.0.0'", "built for torch 1.0.0"), ("_fast_call.py", b"", "no attribute 'torch_version'")])
def test_the_library_alone_serves(tmp_path, module, content, reason):
    """Without the extension module, or with one that does not load or fits another torch: a warning, and every call the Python way."""
    binding.load_library()
    here, there = os.path.dirname(binding.__file__), tmp_path / "paper_2510_08431_amd"
    there.mkdir()
    for name in ("__init__.py", "binding.py", "libattn_jvp.so"):
        os.symlink(os.path.join(here, name), there / name)
    if module:
        (there / module).write_bytes(content)
    res = subprocess.run([sys.executable, "-c", CHILD, str(tmp_path)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and reason in res.stdout, res.stdout + res.stderr
