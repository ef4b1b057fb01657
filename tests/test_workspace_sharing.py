"""The binding's cached workspace: host threads that share a stream share it, and the launches of their calls must not alternate."""
import contextlib
import ctypes
import threading
import time
import types

import pytest
import torch

from paper_2510_08431_amd import binding

DEV = "cuda:0"


class Entry:
    """Stands for the library's entry point: launches nothing, takes its time, and notes whether two calls overlap."""

    def __init__(self):
        self.inside, self.most, self.calls = 0, 0, 0

    def __call__(self, *args):
        self.inside += 1
        self.calls += 1
        self.most = max(self.most, self.inside)
        time.sleep(0.01)
        self.inside -= 1
        return 0


def in_threads(*works):
    threads = [threading.Thread(target=w) for w in works]
    [x.start() for x in threads]
    [x.join() for x in threads]


@pytest.fixture
def stubbed(monkeypatch):
    """The Python way on CPU tensors, up to an entry point that is a stub."""
    entry = Entry()
    monkeypatch.setattr(binding, "_lib", types.SimpleNamespace(attn_jvp_fwd_ex=entry, attn_jvp_fwd_static=entry))
    monkeypatch.setattr(binding, "_fast", types.SimpleNamespace(attn=lambda *a: None))
    monkeypatch.setattr(binding, "_check_inputs", lambda q, k, *a: (*q.shape[:3], k.shape[2], q.shape[3]))
    monkeypatch.setattr(binding, "_raw_stream", lambda device: 7)
    monkeypatch.setattr(binding, "_capturing", lambda *a: False)
    monkeypatch.setattr(binding, "_call", lambda device, fn, *a: fn(*a))
    monkeypatch.setattr(binding, "_workspace_bytes", lambda *a: 256)
    monkeypatch.setattr(binding, "_workspaces", {(torch.device("cpu"), s): torch.empty(256, dtype=torch.uint8) for s in (7, 8)})
    return entry


def test_calls_of_threads_on_one_stream_follow_each_other(stubbed):
    x = torch.zeros(1, 1, 8, 64)
    work = lambda: [binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1) for _ in range(3)]
    in_threads(work, work, work)
    assert stubbed.calls == 9 and stubbed.most == 1


def test_calls_that_share_no_workspace_are_not_held_up(stubbed):
    x = torch.zeros(1, 1, 8, 64)
    other = types.SimpleNamespace(cuda_stream=8)
    in_threads(lambda: [binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1) for _ in range(5)],
               lambda: [binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1, stream=other) for _ in range(5)],
               lambda: [binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1, workspace=None) for _ in range(5)])
    assert stubbed.calls == 15 and stubbed.most >= 2


def test_a_call_inside_a_call_of_the_same_thread(stubbed, monkeypatch):
    """A finalizer that runs while the workspace is made may call in turn."""
    x = torch.zeros(1, 1, 8, 64)
    made, depth = binding._workspaces[(torch.device("cpu"), 7)], []

    def workspace(*a):
        if not depth:
            depth.append(1)
            binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1)
        return made

    monkeypatch.setattr(binding, "_workspace", workspace)
    binding.attn_jvp_fwd_ex(x, x, x, x, x, x, 0.1)
    assert stubbed.calls == 2


@pytest.mark.parametrize("pool", [(1, 0), (0, 0), None])
def test_a_captured_call_has_a_workspace_of_its_own(monkeypatch, pool):
    """Neither the cached buffer nor one for later calls; held for good where it is not in a graph's pool, or nobody can say."""
    cpu = torch.device("cpu")
    cached = torch.empty(256, dtype=torch.uint8)
    monkeypatch.setattr(binding, "_workspaces", {(cpu, 7): cached})
    monkeypatch.setattr(binding, "_kept", [])
    monkeypatch.setattr(binding, "_raw_stream", lambda device: 7)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: None)
    monkeypatch.setattr(torch.cuda, "stream", lambda stream: contextlib.nullcontext())
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)

    def snapshot():
        if pool is None:
            raise RuntimeError("no snapshot")
        return [{"address": 0, "total_size": 1 << 62, "segment_pool_id": pool}]

    monkeypatch.setattr(torch.cuda, "memory_snapshot", snapshot)
    a, b = binding._workspace(cpu, None, 7, 100), binding._workspace(cpu, None, 7, 100)
    assert len({x.data_ptr() for x in (a, b, cached)}) == 3 and binding._workspaces == {(cpu, 7): cached}
    assert len(binding._kept) == (0 if pool == (1, 0) else 2)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    assert binding._workspace(cpu, None, 7, 100) is cached


def inputs(seed, dtype, H, Lq, Lkv, d):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randn(1, H, Lq if i in (0, 3) else Lkv, d, generator=g, device=DEV).to(dtype) for i in range(6)]


@pytest.mark.gpu
def test_native_and_python_calls_of_threads_on_one_stream_follow_each_other(monkeypatch):
    lib = binding.load_library()
    t = inputs(1, torch.float32, 1, 300, 1024, 128)
    entry = Entry()
    prototype = ctypes.CFUNCTYPE(ctypes.c_int, *lib.attn_jvp_fwd_ex.argtypes[:-1], ctypes.c_void_p)
    stub = prototype(entry)
    monkeypatch.setattr(binding, "_lib", types.SimpleNamespace(
        attn_jvp_fwd_ex=entry, attn_jvp_rmsnorm_fwd=lib.attn_jvp_rmsnorm_fwd, attn_jvp_workspace_bytes=lib.attn_jvp_workspace_bytes,
        attn_jvp_workspace_bytes_fp32=lib.attn_jvp_workspace_bytes_fp32))
    try:
        binding._hand_over(binding._fast, lib, stub)
        assert binding._fast.attn(*t, 0.1, torch.float32, 0, 0, 0, True) is not None
        stream = torch.cuda.current_stream()
        in_threads(lambda: [binding.attn_jvp_fwd_ex(*t, 0.1) for _ in range(4)],
                   lambda: [binding.attn_jvp_fwd_ex(*t, 0.1) for _ in range(4)],
                   lambda: [binding.attn_jvp_fwd_ex(*t, 0.1, stream=stream) for _ in range(4)])
    finally:
        binding._hand_over(binding._fast, lib, lib.attn_jvp_fwd_ex)
    assert entry.calls == 13 and entry.most == 1


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,H,Lq,Lkv", [(torch.float32, 1, 300, 1024), (torch.bfloat16, 2, 300, 2300), (torch.bfloat16, 12, 1100, 2100)],
                         ids=["fp32-parts", "bf16-parts", "fp16-values"])
def test_threads_on_one_stream_get_their_own_results(dtype, H, Lq, Lkv):
    sets = [inputs(s, dtype, H, Lq, Lkv, 128) for s in (2, 3, 4)]
    want = [binding.attn_jvp_fwd_ex(*t, 0.1) for t in sets]
    torch.cuda.synchronize()
    got = [[] for _ in sets]

    def work(i):
        got[i].extend(binding.attn_jvp_fwd_ex(*sets[i], 0.1) for _ in range(30))

    in_threads(*[lambda i=i: work(i) for i in range(len(sets))])
    torch.cuda.synchronize()
    for outs, w in zip(got, want):
        assert len(outs) == 30 and all(torch.equal(a, b) for o in outs for a, b in zip(o, w))


@pytest.mark.gpu
@pytest.mark.parametrize("python_way", [False, True], ids=["native", "python"])
@pytest.mark.parametrize("dtype,H,Lq,Lkv", [(torch.float32, 1, 300, 1024), (torch.bfloat16, 2, 300, 2300), (torch.bfloat16, 12, 1100, 2100)],
                         ids=["fp32-parts", "bf16-parts", "fp16-values"])
def test_a_graph_and_what_else_uses_its_stream(dtype, H, Lq, Lkv, python_way):
    """Warmed up, captured and followed by a larger call, all on one stream; replayed with tensors where a freed buffer would be."""
    t, larger = inputs(5, dtype, H, Lq, Lkv, 128), inputs(6, dtype, H, Lq + 500, Lkv, 128)
    side = torch.cuda.Stream()
    kw = {"stream": side} if python_way else {}
    key = (torch.device(DEV), side.cuda_stream)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        want = binding.attn_jvp_fwd_ex(*t, 0.1, **kw)
    torch.cuda.synchronize()
    kept = len(binding._kept)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        got = binding.attn_jvp_fwd_ex(*t, 0.1, **kw)
    assert len(binding._kept) == kept
    cached = binding._workspaces[key]
    cached.fill_(0x5a)
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    assert (cached == 0x5a).all()
    n = cached.numel()
    del cached
    with torch.cuda.stream(side):
        big = binding.attn_jvp_fwd_ex(*larger, 0.1, **kw)
        others = [torch.full((n,), 0x5a, dtype=torch.uint8, device=DEV) for _ in range(3)]
    torch.cuda.synchronize()
    for _ in range(3):
        for x in got:
            x.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want)) and all((x == 0x5a).all() for x in others)
    with torch.cuda.stream(side):
        assert all(torch.equal(a, b) for a, b in zip(big, binding.attn_jvp_fwd_ex(*larger, 0.1, **kw)))


@pytest.mark.gpu
def test_two_graphs_replayed_on_two_streams():
    sets = [inputs(s, torch.float32, 1, 300, 2048, 128) for s in (7, 8)]
    want = [binding.attn_jvp_fwd_ex(*t, 0.1) for t in sets]
    torch.cuda.synchronize()
    graphs, outs = [], []
    for t in sets:
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            outs.append(binding.attn_jvp_fwd_ex(*t, 0.1))
    streams = [torch.cuda.Stream() for _ in sets]
    torch.cuda.synchronize()
    for _ in range(10):
        for g, s in zip(graphs, streams):
            with torch.cuda.stream(s):
                g.replay()
    torch.cuda.synchronize()
    for o, w in zip(outs, want):
        assert all(torch.equal(a, b) for a, b in zip(o, w))
