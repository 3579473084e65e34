"""Performance cases of the framework: what a program that runs a decoder layer shard-invariantly asks of it.

Shapes are those of the row- and column-parallel layers that the tests and the benchmark use: an 8B-class layer (hidden
4096, MLP 12288 or 14336, 32 query heads over 8 key/value heads of 128 channels, leaf 256) and a 32B-class layer (hidden
5120, MLP 25600, 40 heads over 8, leaf 128), a vocabulary of 151936, and the fp32 GEMM shape 6144 x 2048.  Batches go from
one token to a prefill of 4096 and are ragged, as batches of requests are.

The results are compared exactly: the summation order of every kernel is fixed by the method (one binary tree over the
reduction dimension, fixed key tiles and splits in attention), so the bits of a result do not depend on the kernel, the tile
or the launch that computes it.
"""
import math

import torch

from paper_2511_17826_amd import binding as tb

DEV = "cuda"
VOCAB = 151936

# (K, N, leaf, k_first) of the GEMMs of the two layer classes: o_proj and down_proj (row-parallel), qkv (column-parallel)
GEMMS_16 = [(4096, 4096, 256, 1), (12288, 4096, 256, 3), (14336, 4096, 256, 7), (4096, 6144, 256, 1),
            (5120, 5120, 128, 5), (5120, 7168, 128, 5), (25600, 5120, 128, 25)]
GEMMS_LOWBIT = [(4096, 4096, 256, 1), (12288, 4096, 256, 3), (4096, 6144, 256, 1)]
GEMMS_F32 = [(6144, 2048, 128, 3), (4096, 4096, 128, 1), (4096, 4096, 256, 1)]
SWIGLU = [(4096, 12288, 256, 1), (4096, 14336, 256, 1)]                    # (K, I, leaf, k_first)


def listed():
    return [
        # One token through an o_proj-sized layer: the smallest decode step, latency and launches.
        dict(name="gemm_one_token", kind="gemm", dtype="bf16", M=1, K=4096, N=4096, leaf=256, k_first=1, out="same", norm=False),
        # A decode batch of odd size through down_proj in fp16: the weight is read once for all of it.
        dict(name="gemm_decode_batch", kind="gemm", dtype="fp16", M=77, K=12288, N=4096, leaf=256, k_first=3, out="same", norm=False),
        # RMSNorm and the qkv projection of a prefill chunk: the matrix product at full size.
        dict(name="norm_qkv_prefill", kind="gemm", dtype="bf16", M=4096, K=4096, N=6144, leaf=256, k_first=1, out="same", norm=True),
        # The MLP's first half (gate/up projection and the gated activation) of a ragged mid-size batch.
        dict(name="swiglu_mid", kind="swiglu", dtype="bf16", M=500, K=4096, I=12288, leaf=256, k_first=1),
        # The row-parallel layer of a tensor-parallel group of four emulated on one GPU: the shards' partial sums, then
        # the fused tail (tree over the shards, residual, RMSNorm), down_proj at a prefill of 1000 tokens.
        dict(name="tp4_down_proj_tail", kind="tp", dtype="bf16", M=1000, K=12288, N=4096, leaf=256, k_first=3, P=4),
        # A decode batch on an 8-bit weight.
        dict(name="fp8_decode_batch", kind="fp8", fmt="e4m3", M=16, K=12288, N=4096, leaf=256, k_first=3),
        # A prefill on microscaled operands.
        dict(name="mxfp4_prefill", kind="mxfp4", fmt="e2m1", M=4096, K=12288, N=4096, leaf=256, k_first=3),
        dict(name="mxfp8_prefill", kind="mxfp8", fmt="e4m3", M=1500, K=4096, N=4096, leaf=256, k_first=1),
        # Full-precision GEMM on the fp32 shape, ragged rows.
        dict(name="gemm_f32", kind="f32", M=600, K=6144, N=2048, leaf=128, k_first=3),
        # Log-probabilities of a decode batch.
        dict(name="logsoftmax_batch", kind="rows", op="logsoftmax", dtype="fp32", M=48, V=VOCAB),
        # Prefill of four prompts of different lengths.
        dict(name="attention_prefill", kind="attention", dtype="bf16", heads=32, kv_heads=8,
             q_lens="4096,1531,2777,3600", k_lens="4096,1531,2777,3600"),
        # A decode step of a small batch of requests, each at its own context length.
        dict(name="attention_decode", kind="attention", dtype="bf16", heads=32, kv_heads=8,
             q_lens="1,1,1,1,1,1", k_lens="3071,517,1400,2222,4001,96"),
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; odd values as likely as even ones."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def _draw_once(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "swiglu", "tp", "fp8", "mx", "mx", "f32", "rows", "norm", "attention_prefill",
                       "attention_decode", "attention_decode", "attention_mixed"])
    dt = rng.choice(["bf16", "bf16", "fp16"])
    if kind == "gemm":
        K, N, leaf, kf = rng.choice(GEMMS_16)
        return dict(kind="gemm", dtype=dt, M=_log_int(rng, 1, 4096), K=K, N=N, leaf=leaf, k_first=kf,
                    out=rng.choice(["same", "same", "fp32"]), norm=rng.random() < 0.3)
    if kind == "swiglu":
        K, I, leaf, kf = rng.choice(SWIGLU)
        return dict(kind="swiglu", dtype=dt, M=_log_int(rng, 1, 2048), K=K, I=I, leaf=leaf, k_first=kf)
    if kind == "tp":
        K, N, leaf, kf = rng.choice([g for g in GEMMS_16 if g[0] != 4096 or g[1] == 4096])
        return dict(kind="tp", dtype=dt, M=_log_int(rng, 1, 2048), K=K, N=N, leaf=leaf, k_first=kf, P=rng.choice([2, 4, 8]))
    if kind == "fp8":
        K, N, leaf, kf = rng.choice(GEMMS_LOWBIT)
        return dict(kind="fp8", fmt=rng.choice(["e4m3", "e4m3", "e5m2"]), M=_log_int(rng, 1, 4096), K=K, N=N, leaf=leaf, k_first=kf)
    if kind == "mx":
        K, N, leaf, kf = rng.choice(GEMMS_LOWBIT)
        kind, fmt = rng.choice([("mxfp4", "e2m1"), ("mxfp8", "e4m3"), ("mxfp6", "e2m3"), ("mxfp6", "e3m2")])
        return dict(kind=kind, fmt=fmt, M=_log_int(rng, 1, 4096), K=K, N=N, leaf=leaf, k_first=kf)
    if kind == "f32":
        K, N, leaf, kf = rng.choice(GEMMS_F32)
        return dict(kind="f32", M=_log_int(rng, 1, 1500), K=K, N=N, leaf=leaf, k_first=kf)
    if kind == "rows":
        op = rng.choice(["logsoftmax", "logsoftmax", "logsoftmax", "sum", "max"])
        return dict(kind="rows", op=op, dtype=rng.choice(["fp32", "fp32", "bf16", "fp16"]), M=_log_int(rng, 1, 400),
                    V=rng.choice([VOCAB, VOCAB, 32000, 128256, 8 * rng.randrange(500, 1000)]))
    if kind == "norm":
        return dict(kind="norm", dtype=dt, M=_log_int(rng, 1, 8192), H=rng.choice([4096, 5120]))
    heads = rng.choice([32, 32, 40])
    if kind == "attention_prefill":
        n = rng.randrange(1, 5)
        lens = [_log_int(rng, 16, 6000) for _ in range(n)]
        return dict(kind="attention", dtype=dt, heads=heads, kv_heads=8, q_lens=",".join(map(str, lens)), k_lens=",".join(map(str, lens)))
    if kind == "attention_decode":
        n = _log_int(rng, 1, 48)
        longest = _log_int(rng, 128, 16384)
        lens = [_log_int(rng, max(1, longest // 16), longest) for _ in range(n)]
        return dict(kind="attention", dtype=dt, heads=heads, kv_heads=8, q_lens=",".join(["1"] * n), k_lens=",".join(map(str, lens)))
    # decode steps beside one chunk of a prefill
    n = _log_int(rng, 1, 24)
    lens = [_log_int(rng, 32, 4096) for _ in range(n)]
    chunk = _log_int(rng, 64, 1024)
    return dict(kind="attention", dtype=dt, heads=heads, kv_heads=8, q_lens=",".join(["1"] * n + [str(chunk)]),
                k_lens=",".join(map(str, lens + [chunk + _log_int(rng, 1, 4096)])))


def _cost(case):
    """Rough seconds of a pass at rates of this GPU, only to keep the drawn cases below the largest listed one."""
    w = work(case)
    rate = {"f32": 0.1e15, "fp8": 1.8e15, "mxfp8": 1.8e15, "mxfp6": 1.5e15, "mxfp4": 2.4e15}.get(case["kind"], 0.8e15)
    return max(w["bytes"] / 5e12, w["flops"] / rate)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        case = _draw_once(rng)
        if _cost(case) <= most:
            return case


# ---- inputs ----

_TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}


def _randn(g, shape, scale=1.0):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).mul_(scale)


def _block_scales(a, top):
    """E8M0 scale bytes of blocks of 32: the power of two that brings a block's largest magnitude into (top / 2, top]."""
    m = a.view(a.shape[0], -1, 32).abs().amax(dim=2).clamp_(min=2.0 ** -100)
    e = torch.ceil(torch.log2(m / top))
    return e, (e + 127).to(torch.uint8)


def _mx_scaled(a, top):
    e, s = _block_scales(a, top)
    return (a.view(a.shape[0], -1, 32) * torch.exp2(-e).unsqueeze(2)).view_as(a), s


def _nearest(a, values):
    """Index of the nearest of the ascending non-negative `values` for |a|, and the sign bit."""
    v = torch.tensor(values, device=a.device, dtype=torch.float32)
    return torch.bucketize(a.abs(), (v[1:] + v[:-1]) * 0.5).to(torch.uint8), (a < 0).to(torch.uint8)


def _mxfp4(a):
    x, s = _mx_scaled(a, 6.0)
    code, sign = _nearest(x, [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0])
    c = (code | (sign << 3)).view(a.shape[0], -1, 2)
    return (c[:, :, 0] | (c[:, :, 1] << 4)).contiguous(), s


def _mxfp6(a, fmt):
    exp_bits, man, bias, top = (2, 3, 1, 7.5) if fmt == "e2m3" else (3, 2, 3, 28.0)
    values = []
    for p in range(32):
        e, m = p >> man, p & ((1 << man) - 1)
        values.append(m / (1 << man) * 2.0 ** (1 - bias) if e == 0 else (1 + m / (1 << man)) * 2.0 ** (e - bias))
    x, s = _mx_scaled(a, top)
    code, sign = _nearest(x, values)
    c = (code | (sign << 5)).view(a.shape[0], -1, 4)                       # four elements are three bytes, little-endian
    b = torch.stack([c[..., 0] | (c[..., 1] << 6), (c[..., 1] >> 2) | (c[..., 2] << 4), (c[..., 2] >> 4) | (c[..., 3] << 2)], dim=-1)
    return b.view(a.shape[0], -1).contiguous(), s


def _fp8(a, fmt):
    t = torch.float8_e4m3fn if fmt == "e4m3" else torch.float8_e5m2
    top = 448.0 if fmt == "e4m3" else 57344.0
    return a.clamp(-top, top).to(t).view(torch.uint8)


def _mxfp8(a, fmt):
    x, s = _mx_scaled(a, 448.0 if fmt == "e4m3" else 57344.0)
    return _fp8(x, fmt), s


def _quantized(g, rows, K, scale, kind, fmt):
    """A matrix of the low-bit kind in pieces of rows, so that its fp32 form is never whole."""
    parts = []
    for r in range(0, rows, 2048):
        a = _randn(g, (min(2048, rows - r), K), scale)
        q = _mxfp4(a) if kind == "mxfp4" else _mxfp6(a, fmt) if kind == "mxfp6" else _mxfp8(a, fmt)
        parts.append(q)
    return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    kind = case["kind"]
    s = {"case": case}
    if kind in ("gemm", "tp", "swiglu"):
        t = _TORCH[case["dtype"]]
        M, K = case["M"], case["K"]
        N = 2 * case["I"] if kind == "swiglu" else case["N"]
        s["X"] = _randn(g, (M, K)).to(t)
        s["W"] = _randn(g, (K, N), 0.02).to(t)
        if kind == "gemm" and case["norm"]:
            s["norm"] = (1.0 + _randn(g, (K,), 0.1)).to(t)
        if kind == "tp":
            s["norm"] = (1.0 + _randn(g, (N,), 0.1)).to(t)
            s["residual"] = _randn(g, (M, N)).to(t)
    elif kind == "fp8":
        s["X"] = _fp8(_randn(g, (case["M"], case["K"])), case["fmt"])
        s["W"] = _fp8(_randn(g, (case["N"], case["K"])), case["fmt"])      # weights are scaled up to the format's range
    elif kind in ("mxfp4", "mxfp6", "mxfp8"):
        s["X"], s["Xs"] = _quantized(g, case["M"], case["K"], 1.0, kind, case["fmt"])
        s["W"], s["Ws"] = _quantized(g, case["N"], case["K"], 0.02, kind, case["fmt"])
    elif kind == "f32":
        s["X"] = _randn(g, (case["M"], case["K"]))
        s["W"] = _randn(g, (case["K"], case["N"]), 0.02)
    elif kind == "rows":
        s["x"] = _randn(g, (case["M"], case["V"]), 3.0).to(_TORCH[case["dtype"]])
    elif kind == "norm":
        t = _TORCH[case["dtype"]]
        s["x"] = _randn(g, (case["M"], case["H"])).to(t)
        s["norm"] = (1.0 + _randn(g, (case["H"],), 0.1)).to(t)
    elif kind == "attention":
        t = _TORCH[case["dtype"]]
        ql = [int(v) for v in case["q_lens"].split(",")]
        kl = [int(v) for v in case["k_lens"].split(",")]
        s["Q"] = _randn(g, (sum(ql), case["heads"], 128)).to(t)
        s["K"] = _randn(g, (sum(kl), case["kv_heads"], 128)).to(t)
        s["V"] = _randn(g, (sum(kl), case["kv_heads"], 128)).to(t)
        cum = lambda v: torch.tensor([0] + v, dtype=torch.int64).cumsum(0).to(torch.int32).to(DEV)
        s["cu_q"], s["cu_k"], s["max_q"], s["max_k"] = cum(ql), cum(kl), max(ql), max(kl)      # a scheduler knows its lengths
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "gemm":
        f16 = c["dtype"] == "fp16"
        x = s["X"]
        if c["norm"]:
            x = (tb.tbik_rmsnorm_f16 if f16 else tb.tbik_rmsnorm)(x, s["norm"], 1e-6)
        out = torch.float32 if c["out"] == "fp32" else x.dtype
        return (tb.tbik_gemm_f16 if f16 else tb.tbik_gemm)(x, s["W"], c["leaf"], c["k_first"], out_dtype=out)
    if kind == "swiglu":
        return tb.tbik_gemm_swiglu(s["X"], s["W"], c["leaf"], c["k_first"])
    if kind == "tp":
        f16 = c["dtype"] == "fp16"
        parts = (tb.tbik_gemm_shard_partials_f16 if f16 else tb.tbik_gemm_shard_partials)(s["X"], s["W"], c["leaf"], c["k_first"], c["P"])
        tail = tb.tbik_combine_residual_rmsnorm_f16 if f16 else tb.tbik_combine_residual_rmsnorm
        return tail(parts, s["residual"], s["norm"], 1e-6)
    if kind == "fp8":
        return tb.tbik_gemm_fp8(s["X"], s["W"], c["leaf"], c["k_first"], c["fmt"])
    if kind == "mxfp4":
        return tb.tbik_gemm_mxfp4(s["X"], s["Xs"], s["W"], s["Ws"], c["leaf"], c["k_first"])
    if kind == "mxfp6":
        return tb.tbik_gemm_mxfp6(s["X"], s["Xs"], s["W"], s["Ws"], c["leaf"], c["k_first"], c["fmt"])
    if kind == "mxfp8":
        return tb.tbik_gemm_mxfp8(s["X"], s["Xs"], s["W"], s["Ws"], c["leaf"], c["k_first"], c["fmt"])
    if kind == "f32":
        return tb.tbik_gemm_f32(s["X"], s["W"], c["leaf"], c["k_first"])
    if kind == "rows":
        return tb.tbik_row_reduce(s["x"], {"sum": tb.TBIK_SUM, "max": tb.TBIK_MAX, "logsoftmax": tb.TBIK_LOGSOFTMAX}[c["op"]])
    if kind == "norm":
        return (tb.tbik_rmsnorm_f16 if c["dtype"] == "fp16" else tb.tbik_rmsnorm)(s["x"], s["norm"], 1e-6)
    attention = tb.tbik_attention_f16 if c["dtype"] == "fp16" else tb.tbik_attention
    return attention(s["Q"], s["K"], s["V"], s["cu_q"], s["cu_k"], s["max_q"], 128 ** -0.5, causal=True, max_seqlen_k=s["max_k"])


def work(case):
    """Each input read once, each output written once; multiplications and additions counted separately."""
    kind = case["kind"]
    size = {"bf16": 2, "fp16": 2, "fp32": 4}.get(case.get("dtype"), 4)
    if kind == "gemm":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": 2 * (M * K + K * N) + (4 if case["out"] == "fp32" else 2) * M * N, "flops": 2 * M * K * N}
    if kind == "swiglu":
        M, K, I = case["M"], case["K"], case["I"]
        return {"bytes": 2 * (M * K + K * 2 * I + M * I), "flops": 4 * M * K * I}
    if kind == "tp":                                   # a shard's partial sums cross the wire in fp32: written and read once
        M, K, N, P = case["M"], case["K"], case["N"], case["P"]
        return {"bytes": 2 * (M * K + K * N) + 8 * P * M * N + 6 * M * N, "flops": 2 * M * K * N}
    if kind in ("fp8", "mxfp4", "mxfp6", "mxfp8"):
        M, K, N = case["M"], case["K"], case["N"]
        per = {"fp8": 1.0, "mxfp4": 0.5 + 1 / 32, "mxfp6": 0.75 + 1 / 32, "mxfp8": 1 + 1 / 32}[kind]
        return {"bytes": per * (M * K + K * N) + 2 * M * N, "flops": 2 * M * K * N}
    if kind == "f32":
        M, K, N = case["M"], case["K"], case["N"]
        return {"bytes": 4 * (M * K + K * N + M * N), "flops": 2 * M * K * N}
    if kind == "rows":
        M, V = case["M"], case["V"]
        return {"bytes": size * M * V + (4 * M * V if case["op"] == "logsoftmax" else 4 * M), "flops": M * V}
    if kind == "norm":
        return {"bytes": 2 * size * case["M"] * case["H"], "flops": 4 * case["M"] * case["H"]}
    ql = [int(v) for v in case["q_lens"].split(",")]
    kl = [int(v) for v in case["k_lens"].split(",")]
    visible = sum(q * (k - q) + q * (q + 1) // 2 for q, k in zip(ql, kl))              # causal (query, key) pairs
    return {"bytes": 2 * 128 * (2 * case["heads"] * sum(ql) + 2 * case["kv_heads"] * sum(kl)), "flops": 4 * 128 * case["heads"] * visible}


def tolerance(case):
    return "exact"
