"""Performance cases of the attention forward + JVP library.

A case is a dict of plain values.  `listed()` holds the shapes a consistency-distillation program has the library do,
from one small head to the 720p video sequence; `draw(rng)` gives more cases of the same ranges.  Every pass goes
through the public Python entry points (`attn_jvp_fwd_ex`, `attn_jvp_fwd`, `attn_jvp_fwd_static`,
`attn_jvp_rmsnorm_fwd`).

Attention case: B, H, Lq, Lkv, d; dtype "bf16" | "fp32"; tangents "all" (tq, tk, tv), "query" (tk = tv = None) or
"none" (plain forward); gain (factor on q and k after drawing: the scaled logits have standard deviation gain^2);
unit_rms (q, k rows divided by their RMS, as QK-normalisation leaves them); tstd (tangent standard deviation);
blhd (tensors are [B, L, H, d]); out "fp32" | "input"; entry "ex" | "fwd" | "static".
Normalisation case: rows, d, dtype.
"""
import math

import numpy as np
import torch

from paper_2510_08431_amd import attn_jvp_fwd, attn_jvp_fwd_ex, attn_jvp_fwd_static, attn_jvp_rmsnorm_fwd
from paper_2510_08431_amd.binding import LAYOUT_BHLD, LAYOUT_BLHD

_DTYPE = {"bf16": torch.bfloat16, "fp32": torch.float32}
_SIZE = {"bf16": 2, "fp32": 4}
_EPS = 1e-6


def _attn(name, B, H, Lq, Lkv, d, dtype="bf16", tangents="all", gain=1.0, unit_rms=False, tstd=0.5, blhd=False,
          out="fp32", entry="ex"):
    return {"name": name, "op": "attn", "B": B, "H": H, "Lq": Lq, "Lkv": Lkv, "d": d, "dtype": dtype,
            "tangents": tangents, "gain": gain, "unit_rms": unit_rms, "tstd": tstd, "blhd": blhd, "out": out,
            "entry": entry}


def listed():
    return [
        # the smallest self-attention block, in fp32: two heads of 256 tokens (workload 1)
        _attn("tiny-self-fp32", 1, 2, 256, 256, 64, "fp32", tstd=1.0),
        # a small conditioning block: 300 image tokens onto a ragged 77-token context without tangents; latency
        _attn("small-cross-bf16", 1, 8, 300, 77, 64, tangents="query"),
        # one latent frame of the 480p video (32760 = 21 x 1560 tokens): ragged query and key tails, bf16 outputs
        _attn("frame-self-bf16", 1, 12, 1560, 1560, 128, unit_rms=True, out="input"),
        # image diffusion transformer, self-attention behind QK-normalisation (workload 2)
        _attn("image-self-bf16", 2, 16, 4096, 4096, 128, unit_rms=True),
        # the same block run in fp32 (bench.py --config 2 --input-dtype fp32)
        _attn("image-self-fp32", 2, 16, 4096, 4096, 128, "fp32", unit_rms=True),
        # the same block without tangents: a teacher's or sampler's plain forward, bf16 outputs
        _attn("image-plain-bf16", 2, 16, 4096, 4096, 128, tangents="none", unit_rms=True, out="input"),
        # a sequence of 5000 tokens at a head dimension between the two usual ones, whole call on the library's own scratch
        _attn("self-d96-bf16", 1, 12, 5000, 5000, 96, entry="static"),
        # video self-attention, 12 heads x 32760 tokens (workload 3)
        _attn("video-self-bf16", 1, 12, 32760, 32760, 128),
        # video cross-attention onto 512 text tokens that carry no tangent (workload 4)
        _attn("video-cross-bf16", 1, 12, 32760, 512, 128, tangents="query"),
        # the video shape at head dimension 64, same model width (workload 6)
        _attn("video-self-d64-bf16", 1, 24, 32760, 32760, 64),
        # 720p video of the 14B model, one of eight context-parallel shards (5 of 40 heads, as the sequence-to-head
        # all-to-all leaves them), peaked rows: logit standard deviation 8 (workload 5)
        _attn("video-720p-shard-bf16", 1, 5, 75600, 75600, 128, gain=math.sqrt(8.0), tstd=1.0, blhd=True, out="input"),
        # QK-normalisation of the video sequence's queries, 12 heads x 32760 rows
        {"name": "qk-norm-video-bf16", "op": "norm", "rows": 393120, "d": 128, "dtype": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.12:
        return {"op": "norm", "rows": _log_int(rng, 300, 400000), "d": rng.choice([64, 128, 128, 256]),
                "dtype": rng.choice(["bf16", "bf16", "fp32"])}
    d = rng.choice([32, 64, 64, 96, 128, 128, 128, 256])
    dtype = rng.choice(["bf16", "bf16", "fp32"])
    tangents = rng.choice(["all", "all", "all", "query", "none"])
    # counted operations of a drawn case: what the path does in at most some 30 ms, far below the largest listed case
    most = 5e10 if d == 256 else 8e11 if dtype == "fp32" else 8e12
    B, H = rng.choice([1, 1, 2, 4]), rng.randint(1, 24)
    if tangents == "query":                       # cross-attention
        Lq, Lkv = _log_int(rng, 64, 32760), _log_int(rng, 16, 1024)
    else:
        Lq = Lkv = _log_int(rng, 64, 32760)
    while 12.0 * B * H * Lq * Lkv * d > most:
        if B > 1:
            B //= 2
        elif H > 1:
            H = (H + 1) // 2
        else:
            Lq = max(64, Lq * 2 // 3)
            Lkv = max(16, Lkv * 2 // 3)
    blhd = rng.random() < 0.25
    out = rng.choice(["fp32", "fp32", "input"])
    entry = "ex"
    if dtype == "bf16" and d in (64, 128) and not blhd and out == "fp32":
        entry = rng.choice(["ex", "ex", "fwd"])
    gain = rng.choice([1.0, 1.0, 1.0, math.sqrt(2.0), math.sqrt(8.0)])
    case = _attn("", B, H, Lq, Lkv, d, dtype, tangents, gain, rng.random() < 0.5, rng.choice([0.5, 1.0]), blhd, out, entry)
    del case["name"]
    return case


def _scale(case):
    return float(np.float32(case["d"] ** -0.5))      # the C interface takes a float: a value that it holds exactly


def _make_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)

    if case["op"] == "norm":
        dt, n, d = _DTYPE[case["dtype"]], case["rows"], case["d"]
        return {"x": (1.5 * normal(n, d)).to(dt), "tx": (0.5 * normal(n, d)).to(dt), "w": 1.0 + 0.1 * normal(d)}
    B, H, d, dt = case["B"], case["H"], case["d"], _DTYPE[case["dtype"]]
    t = {}
    for name in ("q", "k", "v", "tq", "tk", "tv"):
        if (name == "tq" and case["tangents"] == "none") or (name in ("tk", "tv") and case["tangents"] != "all"):
            t[name] = None
            continue
        L = case["Lq"] if name in ("q", "tq") else case["Lkv"]
        x = normal(B, L, H, d) if case["blhd"] else normal(B, H, L, d)
        if name in ("q", "k"):
            if case["unit_rms"]:
                x = x / x.pow(2).mean(dim=-1, keepdim=True).sqrt()
            x = x * case["gain"]
        elif name != "v":
            x = x * case["tstd"]
        t[name] = x.to(dt)
        del x
    return t


def prepare(case, seed):
    state = _make_inputs(case, seed)
    state["case"] = case
    if case["op"] == "attn":
        state["scale"] = _scale(case)
        if case["entry"] == "static":      # this entry point writes into outputs that the program brings
            q = state["q"]
            o = torch.empty(q.shape, device="cuda", dtype=torch.float32 if case["out"] == "fp32" else q.dtype)
            to = None if state["tq"] is None else torch.empty_like(o)
            state["outputs"] = (o, to, torch.empty(case["B"], case["H"], case["Lq"], device="cuda", dtype=torch.float32))
    return state


def run(state):
    case = state["case"]
    if case["op"] == "norm":
        return attn_jvp_rmsnorm_fwd(state["x"], state["tx"], state["w"], _EPS)
    args = [state[n] for n in ("q", "k", "v", "tq", "tk", "tv")]
    if case["entry"] == "fwd":
        o, to, lse = attn_jvp_fwd(*args, state["scale"])
    elif case["entry"] == "static":
        o, to, lse = attn_jvp_fwd_static(*args, state["scale"], state["outputs"])
    else:
        o, to, lse = attn_jvp_fwd_ex(*args, state["scale"],
                                     out_dtype=torch.float32 if case["out"] == "fp32" else args[0].dtype,
                                     layout=LAYOUT_BLHD if case["blhd"] else LAYOUT_BHLD)
    return (o, lse) if to is None else (o, to, lse)


def work(case):
    if case["op"] == "norm":
        n = case["rows"] * case["d"]
        return {"bytes": 4 * n * _SIZE[case["dtype"]] + 4 * case["d"], "flops": 10 * n}
    B, H, Lq, Lkv, d = (case[n] for n in ("B", "H", "Lq", "Lkv", "d"))
    size = _SIZE[case["dtype"]]
    # products of 2 Lq Lkv d operations: S, tQ K^T, Q tK^T, P V, H V, P tV
    products = {"all": 6, "query": 4, "none": 2}[case["tangents"]]
    q_like = 1 if case["tangents"] == "none" else 2
    kv_like = 4 if case["tangents"] == "all" else 2
    out_size = 4 if case["out"] == "fp32" else size
    rows = B * H * Lq
    return {"bytes": rows * d * q_like * (size + out_size) + 4 * rows + B * H * Lkv * d * kv_like * size,
            "flops": 2 * products * B * H * Lq * Lkv * d}


def tolerance(case):
    # About four times the relative error against 64 bits, as measured over the listed and some drawn cases.
    if case["op"] == "norm":                       # bf16: two roundings to 8 bits (2.4e-3 measured)
        return {"rel": 1e-2 if case["dtype"] == "bf16" else 1e-6}
    if case["dtype"] == "fp32":                    # 32-bit sums over the keys: up to 3.4e-6 measured
        return {"rel": 1.5e-5}
    if case["out"] == "input":                     # the results themselves are rounded to bf16: 1.7e-3 measured
        return {"rel": 7e-3}
    return {"rel": 1.5e-3}                         # 11-bit weights against bf16 values: 3.6e-4 measured


def _exact_norm(t):
    x, tx, w = t["x"].double(), t["tx"].double(), t["w"].double()
    r = (x.pow(2).mean(-1, keepdim=True) + _EPS).rsqrt()
    return x * r * w, (tx * r - x * r.pow(3) * (x * tx).mean(-1, keepdim=True)) * w


def exact(case, seed):
    t = _make_inputs(case, seed)
    if case["op"] == "norm":
        return _exact_norm(t)
    B, H, Lq, Lkv, d = (case[n] for n in ("B", "H", "Lq", "Lkv", "d"))
    scale = _scale(case)

    def head(x, b, h):
        return None if x is None else (x[b, :, h] if case["blhd"] else x[b, h]).double()

    o = torch.empty(t["q"].shape, device="cuda", dtype=torch.float64)
    to = None if t["tq"] is None else torch.empty_like(o)
    lse = torch.empty(B, H, Lq, device="cuda", dtype=torch.float64)
    step = max(1, min(Lq, (1 << 27) // Lkv))          # query rows at a time: 1 GiB per matrix of scores
    for b in range(B):
        for h in range(H):
            q, k, v, tq, tk, tv = (head(t[n], b, h) for n in ("q", "k", "v", "tq", "tk", "tv"))
            oh = o[b, :, h] if case["blhd"] else o[b, h]
            toh = None if to is None else (to[b, :, h] if case["blhd"] else to[b, h])
            for i in range(0, Lq, step):
                rows = slice(i, min(i + step, Lq))
                p = (q[rows] @ k.T).mul_(scale)
                z = torch.logsumexp(p, dim=-1)
                lse[b, h, rows] = z
                p.sub_(z[:, None]).exp_()
                oh[rows] = p @ v
                if to is not None:
                    g = tq[rows] @ k.T
                    if tk is not None:
                        g.addmm_(q[rows], tk.T)
                    g.mul_(scale).mul_(p)                            # P o tS
                    g.sub_(p * g.sum(-1, keepdim=True))              # tP
                    y = g @ v
                    if tv is not None:
                        y.addmm_(p, tv)
                    toh[rows] = y
    return (o, lse) if to is None else (o, to, lse)
