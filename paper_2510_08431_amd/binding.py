"""Binding of the attn_jvp C-ABI library: argument marshalling only, through ctypes, and for the ordinary calls through the
extension module _fast_call (csrc/fast_call.cpp), which does the same steps natively (where it does not load, with a warning,
every call takes the first way).

PyTorch supplies device memory (`data_ptr()`) and the current HIP stream; every step of
the computation runs inside the library's kernels.  There is no CPU or eager fallback:
if the shared library is missing, loading raises.
"""
import contextlib
import ctypes
import functools
import os
import threading
import warnings

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libattn_jvp.so")

KERNEL_AUTO, KERNEL_FP32, KERNEL_MFMA = 0, 1, 2
LAYOUT_BHLD = 0   # tensors are [B, H, L, d]
LAYOUT_BLHD = 1   # tensors are [B, L, H, d] (lse stays [B, H, Lq])
FLAG_FAST = 1     # MFMA kernel: P~ and H~ as single bf16 terms (6 matrix products per key block; not tolerance-safe)
FLAG_F16_ALWAYS = 4   # MFMA kernel: fp16 value path also for short key sequences (given a workspace)
FLAG_NO_LOCKSTEP = 8   # MFMA kernel, running-reference fp16 tier: no lock-step start of the tiles of an XCD
FLAG_NO_RESIDENT = 16   # MFMA kernel: one workgroup per query tile instead of resident workgroups
FLAG_NO_F16 = 2   # MFMA kernel: hi + lo bf16 pairs (9 products) even when a workspace is available
_DTYPE_CODE = {torch.bfloat16: 0, torch.float32: 1}


class AttnJvpOpts(ctypes.Structure):
    _fields_ = [("in_dtype", ctypes.c_int), ("out_dtype", ctypes.c_int), ("stream", ctypes.c_void_p),
                ("kernel", ctypes.c_int), ("flags", ctypes.c_int), ("workspace", ctypes.c_void_p),
                ("workspace_bytes", ctypes.c_size_t), ("timing_events", ctypes.c_void_p * 2),
                ("layout", ctypes.c_int), ("reserved", ctypes.c_int)]


class AttnJvpError(RuntimeError):
    def __init__(self, code, message):
        super().__init__(f"attn_jvp error {code}: {message}")
        self.code = code


class _NoFastCall:
    """In the extension module's place where it cannot be used: no call is an ordinary one."""
    attn = rmsnorm = staticmethod(lambda *a: None)


_lib = None
_fast = None      # the extension module, once the library is loaded
_AUTO = "auto"


def load_library():
    """Load libattn_jvp.so (built in-tree by __graft_entry__.build()) and declare its symbols."""
    global _lib, _fast
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise FileNotFoundError(
            f"{LIB_PATH} not found: build the HIP library first (python -c 'import __graft_entry__ as g; g.build()')")
    lib = ctypes.CDLL(LIB_PATH)
    vp, ci, cf = ctypes.c_void_p, ctypes.c_int, ctypes.c_float
    common = [vp] * 9 + [ci] * 5 + [cf]
    lib.attn_jvp_fwd.argtypes = common
    lib.attn_jvp_fwd.restype = ci
    lib.attn_jvp_fwd_ex.argtypes = common + [ctypes.POINTER(AttnJvpOpts)]
    lib.attn_jvp_fwd_ex.restype = ci
    lib.attn_jvp_fwd_static.argtypes = common + [ctypes.POINTER(AttnJvpOpts)]
    lib.attn_jvp_fwd_static.restype = ci
    lib.attn_jvp_static_scratch_bytes.argtypes = []
    lib.attn_jvp_static_scratch_bytes.restype = ctypes.c_size_t
    lib.attn_jvp_strerror.argtypes = [ci]
    lib.attn_jvp_strerror.restype = ctypes.c_char_p
    lib.attn_jvp_version.argtypes = []
    lib.attn_jvp_version.restype = ci
    lib.attn_jvp_rmsnorm_fwd.argtypes = [vp] * 5 + [ctypes.c_longlong, ci, ctypes.c_float, ci, vp]
    lib.attn_jvp_rmsnorm_fwd.restype = ci
    lib.attn_jvp_mfma_rate_probe.argtypes = [vp, vp, ci, ci, vp, ctypes.POINTER(ctypes.c_longlong), ctypes.POINTER(ci)]
    lib.attn_jvp_mfma_rate_probe.restype = ci
    lib.attn_jvp_workspace_bytes.argtypes = [ci] * 5
    lib.attn_jvp_workspace_bytes.restype = ctypes.c_size_t
    lib.attn_jvp_workspace_bytes_fp32.argtypes = [ci] * 5
    lib.attn_jvp_workspace_bytes_fp32.restype = ctypes.c_size_t
    lib.attn_jvp_route.argtypes = [ci] * 5 + [cf, ci, ctypes.POINTER(AttnJvpOpts), ctypes.POINTER(ci)]
    lib.attn_jvp_route.restype = ci
    _fast = _load_fast_call()
    if _fast is not _NoFastCall:
        _hand_over(_fast, lib, lib.attn_jvp_fwd_ex)
    _lib = lib
    return lib


def _load_fast_call():
    """The extension module, or _NoFastCall: it only saves host time, and is tied to the torch and Python it was built with."""
    try:
        from . import _fast_call
        if _fast_call.torch_version == torch.__version__:
            return _fast_call
        reason = f"built for torch {_fast_call.torch_version}, this is {torch.__version__}"
    except (ImportError, AttributeError) as e:
        reason = str(e)
    warnings.warn(f"attn_jvp: host time per call is higher without the extension module _fast_call ({reason}); "
                  "build it: python -c 'import __graft_entry__ as g; g.build()'", RuntimeWarning, stacklevel=3)
    return _NoFastCall


def _hand_over(fast, lib, fwd_ex):
    """Give the extension module what it calls: entry points of the library, and this module's workspaces and locks."""
    entries = (fwd_ex, lib.attn_jvp_rmsnorm_fwd, lib.attn_jvp_workspace_bytes, lib.attn_jvp_workspace_bytes_fp32)
    fast.init(*[ctypes.cast(e, ctypes.c_void_p).value for e in entries], _workspaces, _workspace, _workspace_locks, _workspace_lock)


def attn_jvp_strerror(code):
    return load_library().attn_jvp_strerror(int(code)).decode()


def attn_jvp_version():
    return load_library().attn_jvp_version()


def attn_jvp_workspace_bytes(B, H, Lq, Lkv, d):
    return int(load_library().attn_jvp_workspace_bytes(B, H, Lq, Lkv, d))


ROUTES = ("vector", "keysplit", "f32-tiles", "bf16-pairs", "f16-values", "bf16-single")      # ATTN_JVP_ROUTE_*


def attn_jvp_route(B, H, Lq, Lkv, d, scale, dtype=torch.bfloat16, tangents=2, kernel=KERNEL_AUTO, flags=0, workspace="auto"):
    """What attn_jvp_fwd_ex runs for such a call: (one of ROUTES, the parts its keys go in).  tangents: 0 none, 1 the query's,
    2 all; workspace: "auto" or None."""
    opts = AttnJvpOpts(_DTYPE_CODE[dtype], 0, None, int(kernel), int(flags))
    if workspace == "auto":
        opts.workspace_bytes = _workspace_bytes(B, H, Lq, Lkv, d, dtype == torch.float32)
        opts.workspace = 256 if opts.workspace_bytes else None      # (an aligned address; nobody looks there)
    parts = ctypes.c_int(1)
    route = load_library().attn_jvp_route(B, H, Lq, Lkv, d, float(scale), int(tangents), ctypes.byref(opts), ctypes.byref(parts))
    if route < 0:
        raise AttnJvpError(-route, attn_jvp_strerror(-route))
    return ROUTES[route], parts.value


_workspaces = {}
_workspace_locks = {}


def _workspace_lock(key):
    """The lock of one (device, stream)'s cached workspace, held from its look-up until a call's last launch is enqueued: the
    launches of a call hand the workspace on to one another, so those of two threads on one stream must not alternate.  (Both
    ways of calling drop the GIL meanwhile.  Reentrant: a signal handler or finalizer may make a whole call in between.)"""
    return _workspace_locks.setdefault(key, threading.RLock())


@functools.lru_cache(maxsize=1024)
def _workspace_bytes(B, H, Lq, Lkv, d, f32):
    lib = load_library()
    entry = lib.attn_jvp_workspace_bytes_fp32 if f32 else lib.attn_jvp_workspace_bytes
    return int(entry(B, H, Lq, Lkv, d))      # (host arithmetic on the five numbers)


def _workspace(device, stream, raw_stream, nbytes):
    """A scratch tensor from torch's allocator per (device, stream), grown on demand and reused across calls.

    Whole calls enqueued on one stream run in order, so they can share scratch (under _workspace_lock, which the caller holds);
    calls on different streams may overlap and get separate buffers.  Callers that want to own the memory pass their own
    `workspace`.  `stream` may be None: the current one, whose handle raw_stream is."""
    key = (device, raw_stream)
    capturing = _capturing(device, stream, raw_stream)
    ws = None if capturing else _workspaces.get(key)
    if ws is None or ws.numel() < nbytes:
        if stream is None:
            stream = torch.cuda.current_stream(device)
        with torch.cuda.stream(stream):      # so that torch's caching allocator ties the block to this stream
            ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
        if not capturing:
            _workspaces[key] = ws
        elif not _of_a_graph(ws):
            _kept.append(ws)
    return ws


_kept = []


def _capturing(device, stream, raw_stream):
    """Whether the call is recorded into a graph: it then gets a buffer of its own, not the cached one, which a later call may
    replace while the graph still writes to it, and which other graphs and eager calls would share."""
    if raw_stream == 0:      # (the default stream cannot be captured)
        return False
    if device.index == torch.cuda.current_device() and raw_stream == _raw_stream(device):
        return torch.cuda.is_current_stream_capturing()
    with torch.cuda.stream(torch.cuda.current_stream(device) if stream is None else stream):
        return torch.cuda.is_current_stream_capturing()


def _of_a_graph(ws):
    """Whether ws lies in a graph's private pool, whose memory eager work never gets, so that nobody needs to hold it.  (Under a capture
    that torch does not know of it does not, and _kept holds it until the process ends: nobody says when such a graph goes.)"""
    try:
        segments = torch.cuda.memory_snapshot()
    except RuntimeError:      # (an allocator that cannot say)
        return False
    return any(s["address"] <= ws.data_ptr() < s["address"] + s["total_size"] and tuple(s["segment_pool_id"]) != (0, 0) for s in segments)


def _raw_stream(device):
    """Handle of torch's current stream, without the Stream object that torch.cuda.current_stream makes (2 us)."""
    return torch._C._cuda_getCurrentRawStream(device.index)


def _ptr(t):
    return t.data_ptr() if t is not None else None


def _check_inputs(q, k, v, tq, tk, tv, layout=LAYOUT_BHLD):
    qs, ks = q.shape, k.shape
    if len(qs) != 4 or len(ks) != 4:
        raise ValueError("q and k must be [B, H, L, d] (or [B, L, H, d] with layout=LAYOUT_BLHD)")
    if layout == LAYOUT_BLHD:
        B, Lq, H, d = qs
        Lkv = ks[1]
        kv_shape = (B, Lkv, H, d)
    elif layout == LAYOUT_BHLD:
        B, H, Lq, d = qs
        Lkv = ks[2]
        kv_shape = (B, H, Lkv, d)
    else:
        raise ValueError(f"unknown layout {layout}")
    if (tk is None) != (tv is None):
        raise ValueError("tk and tv must both be given or both be None (zero key/value tangents)")
    if tq is None and tk is not None:
        raise ValueError("tq=None means no tangents at all: tk and tv must be None too")
    dtype, device = q.dtype, q.device
    for name, t, shape in (("q", q, qs), ("tq", tq, qs), ("k", k, kv_shape), ("v", v, kv_shape), ("tk", tk, kv_shape), ("tv", tv, kv_shape)):
        if t is None:
            continue
        if t.shape != shape:
            raise ValueError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")
        if t.dtype is not dtype or t.device != device:
            raise ValueError(f"{name}: dtype/device differ from q")
        if not t.is_contiguous():
            raise ValueError(f"{name} must be contiguous")
    if dtype not in _DTYPE_CODE:
        raise ValueError(f"unsupported dtype {dtype}")
    if not q.is_cuda:
        raise ValueError("tensors must live on the GPU; there is no CPU path")
    return B, H, Lq, Lkv, d


def _call(device, fn, *args):
    """fn(*args) with `device` current: the library enqueues on the current device."""
    if torch.cuda.current_device() == device.index:      # (entering the context manager costs 3 us)
        return fn(*args)
    with torch.cuda.device(device):
        return fn(*args)


def attn_jvp_fwd_ex(q, k, v, tq, tk, tv, scale, out=None, out_dtype=torch.float32, kernel=KERNEL_AUTO, stream=None,
                    flags=0, workspace="auto", timing_events=None, layout=LAYOUT_BHLD):
    """Enqueue O, tO, lse = attention forward + JVP on the current (or given) stream.

    q, tq: [B, H, Lq, d]; k, v, tk, tv: [B, H, Lkv, d]; bf16 or fp32, contiguous, on the GPU.  tk and tv may both be
    None: zero key/value tangents (cross-attention onto a context without tangent); tq, tk, tv all None: plain
    attention forward, the returned `to` is None.
    out: optional (o, to, lse) to write into.  workspace: "auto" (a torch buffer cached per device and stream; one of its own for a call that is captured), None (no
    scratch: the kernel then uses its bf16-pair path), a uint8 CUDA tensor, or "static" (the C entry point
    attn_jvp_fwd_static: the library's own static device array; with `out` given the call allocates nothing).  layout=LAYOUT_BLHD: all eight
    tensors are [B, L, H, d] instead (lse stays [B, H, Lq]).  timing_events: optional pair of
    torch.cuda.Event(enable_timing=True) that the library records right before and after the main kernel.
    Returns (o, to, lse); asynchronous.
    """
    lib = _lib or load_library()
    if out is None and stream is None and timing_events is None and (workspace is None or workspace is _AUTO):
        done = _fast.attn(q, k, v, tq, tk, tv, scale, out_dtype, kernel, flags, layout, workspace is _AUTO)
        if done is not None:      # (None: not an ordinary call)
            if type(done) is int:
                raise AttnJvpError(done, attn_jvp_strerror(done))
            return done
    B, H, Lq, Lkv, d = _check_inputs(q, k, v, tq, tk, tv, layout)
    device = q.device
    if out is None:
        o = torch.empty_like(q, dtype=out_dtype, memory_format=torch.contiguous_format)     # same layout as q
        to = torch.empty_like(o) if tq is not None else None
        lse = torch.empty((B, H, Lq), dtype=torch.float32, device=device)
    else:
        o, to, lse = out
        out_dtype = o.dtype
        if (tuple(o.shape) != tuple(q.shape) or tuple(lse.shape) != (B, H, Lq)
                or (to is not None and tuple(to.shape) != tuple(q.shape)) or (to is None and tq is not None)):
            raise ValueError("out must be (o, to, lse) with o, to shaped like q and lse [B, H, Lq]")
    if out_dtype not in (torch.float32, q.dtype):
        raise ValueError("out_dtype must be float32 or the input dtype")
    raw_stream = _raw_stream(device) if stream is None else stream.cuda_stream
    entry = lib.attn_jvp_fwd_ex
    if isinstance(workspace, str) and workspace == "static":
        entry = lib.attn_jvp_fwd_static
        workspace = None
    opts = AttnJvpOpts(_DTYPE_CODE[q.dtype], 0 if out_dtype == torch.float32 else 1, raw_stream, int(kernel), int(flags))
    opts.layout = int(layout)
    if timing_events is not None:
        for i, ev in enumerate(timing_events):
            if not ev.cuda_event:      # torch creates the HIP event lazily, at its first record
                ev.record(torch.cuda.current_stream(device) if stream is None else stream)
            opts.timing_events[i] = ev.cuda_event
    need = 0
    if isinstance(workspace, str) and workspace == "auto":
        need = _workspace_bytes(B, H, Lq, Lkv, d, q.dtype == torch.float32)
        workspace = None
    with _workspace_lock((device, raw_stream)) if need else contextlib.nullcontext():
        if need:
            workspace = _workspace(device, stream, raw_stream, need)
        if workspace is not None:
            opts.workspace = workspace.data_ptr()
            opts.workspace_bytes = workspace.numel() * workspace.element_size()
        rc = _call(device, entry, q.data_ptr(), k.data_ptr(), v.data_ptr(), _ptr(tq), _ptr(tk), _ptr(tv),
                   o.data_ptr(), _ptr(to), lse.data_ptr(), B, H, Lq, Lkv, d, float(scale), ctypes.byref(opts))
    if rc != 0:
        raise AttnJvpError(rc, attn_jvp_strerror(rc))
    return o, to, lse


def attn_jvp_static_scratch_bytes():
    return int(load_library().attn_jvp_static_scratch_bytes())


def attn_jvp_fwd_static(q, k, v, tq, tk, tv, scale, out, **kw):
    """The C entry point `attn_jvp_fwd_static`: as attn_jvp_fwd_ex, with the library's static device scratch in
    place of a workspace.  `out` = (o, to, lse) is required, so that nothing is allocated on the way."""
    if out is None:
        raise ValueError("attn_jvp_fwd_static writes into caller-provided outputs: pass out=(o, to, lse)")
    return attn_jvp_fwd_ex(q, k, v, tq, tk, tv, scale, out=out, workspace="static", **kw)


def attn_jvp_rmsnorm_fwd(x, tx, w, eps, out=None, stream=None):
    """Enqueue y, ty = RMS normalisation with gain w and its JVP over the last dimension.

    x, tx: [..., d] bf16 or fp32, contiguous, on the GPU; w: [d] float32.  out: optional (y, ty) to write into
    (may be (x, tx) themselves).  Returns (y, ty); asynchronous."""
    lib = _lib or load_library()
    if out is None and stream is None:
        done = _fast.rmsnorm(x, tx, w, eps)
        if done is not None:
            if type(done) is int:
                raise AttnJvpError(done, attn_jvp_strerror(done))
            return done
    if x.dtype not in _DTYPE_CODE or tx.dtype != x.dtype or tuple(tx.shape) != tuple(x.shape):
        raise ValueError("x and tx must have the same shape and dtype (bf16 or fp32)")
    if not (x.is_cuda and tx.is_cuda and w.is_cuda):
        raise ValueError("tensors must live on the GPU; there is no CPU path")
    if not (x.is_contiguous() and tx.is_contiguous() and w.is_contiguous()):
        raise ValueError("x, tx and w must be contiguous")
    d = x.shape[-1]
    if w.dtype != torch.float32 or tuple(w.shape) != (d,):
        raise ValueError("w must be a float32 vector of length d")
    rows = x.numel() // d
    if out is None:
        y, ty = torch.empty_like(x), torch.empty_like(tx)
    else:
        y, ty = out
        if y.dtype != x.dtype or ty.dtype != x.dtype or tuple(y.shape) != tuple(x.shape) or tuple(ty.shape) != tuple(x.shape):
            raise ValueError("out must be (y, ty) shaped and typed like x")
    raw_stream = _raw_stream(x.device) if stream is None else stream.cuda_stream
    rc = _call(x.device, lib.attn_jvp_rmsnorm_fwd, x.data_ptr(), tx.data_ptr(), w.data_ptr(), y.data_ptr(), ty.data_ptr(),
               rows, d, float(eps), _DTYPE_CODE[x.dtype], raw_stream)
    if rc != 0:
        raise AttnJvpError(rc, attn_jvp_strerror(rc))
    return y, ty


def attn_jvp_mfma_rate_probe(operands, out, f16, iters, stream=None):
    """Enqueue the library's back-to-back MFMA loop on the operand values given (measurement aid).

    operands: uint8/int tensor of 8 * 256 * 16 bytes on the GPU (bf16 or fp16 bit patterns); out: float32 tensor with
    at least 256 elements per compute unit.  Returns the number of floating-point operations the launch performs;
    the caller times it."""
    lib = load_library()
    if not (operands.is_cuda and out.is_cuda and operands.is_contiguous() and out.is_contiguous()):
        raise ValueError("operands and out must be contiguous GPU tensors")
    if operands.numel() * operands.element_size() < 8 * 256 * 16:
        raise ValueError("operands must hold 8 x 256 x 16 bytes")
    cus = torch.cuda.get_device_properties(out.device).multi_processor_count
    if out.dtype != torch.float32 or out.numel() < 256 * cus:
        raise ValueError("out must be float32 with 256 elements per compute unit")
    if stream is None:
        stream = torch.cuda.current_stream(out.device)
    per_wave, waves = ctypes.c_longlong(0), ctypes.c_int(0)
    with torch.cuda.device(out.device):
        rc = lib.attn_jvp_mfma_rate_probe(operands.data_ptr(), out.data_ptr(), int(bool(f16)), int(iters),
                                          stream.cuda_stream, ctypes.byref(per_wave), ctypes.byref(waves))
    if rc != 0:
        raise AttnJvpError(rc, attn_jvp_strerror(rc))
    return 32768.0 * per_wave.value * waves.value


def attn_jvp_fwd(q, k, v, tq, tk, tv, scale, out=None):
    """The C entry point `attn_jvp_fwd`: bf16 inputs, fp32 outputs, no workspace, the default stream.

    When torch's current stream is not the default stream the same kernel is enqueued there through
    `attn_jvp_fwd_ex` instead (no workspace either)."""
    lib = load_library()
    if out is None and getattr(q, "dtype", None) is torch.bfloat16:
        # (the entry point on the default stream and attn_jvp_fwd_ex without a workspace on the current one are the same call)
        done = _fast.attn(q, k, v, tq, tk, tv, scale, torch.float32, KERNEL_AUTO, 0, LAYOUT_BHLD, False)
        if done is not None:
            if type(done) is int:
                raise AttnJvpError(done, attn_jvp_strerror(done))
            return done
    B, H, Lq, Lkv, d = _check_inputs(q, k, v, tq, tk, tv)
    if q.dtype != torch.bfloat16:
        raise ValueError("attn_jvp_fwd takes bf16 inputs; use attn_jvp_fwd_ex for fp32")
    if _raw_stream(q.device) != 0:
        return attn_jvp_fwd_ex(q, k, v, tq, tk, tv, scale, out=out, workspace=None)
    if out is None:
        o = torch.empty(B, H, Lq, d, dtype=torch.float32, device=q.device)
        to = torch.empty_like(o) if tq is not None else None
        lse = torch.empty(B, H, Lq, dtype=torch.float32, device=q.device)
    else:
        o, to, lse = out
    rc = _call(q.device, lib.attn_jvp_fwd, q.data_ptr(), k.data_ptr(), v.data_ptr(), _ptr(tq), _ptr(tk), _ptr(tv),
               o.data_ptr(), _ptr(to), lse.data_ptr(), B, H, Lq, Lkv, d, float(scale))
    if rc != 0:
        raise AttnJvpError(rc, attn_jvp_strerror(rc))
    return o, to, lse
