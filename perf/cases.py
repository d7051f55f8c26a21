"""The products a user of this framework computes, as timed cases.

Every case goes through the public entry points of ``paper_2210_16691_amd`` with their default
schedule (``sched=None``), into output tensors the caller owns.  The listed sizes are those of
``workloads.CONFIGS`` and the tests, or generic; ``draw`` spreads over the ranges around them.

Kinds of case:

linear           C = A.B, optionally with bias and ReLU in the epilogue, B stored K x N or N x K
attention        the two batched products of self-attention: Q.K^T scaled, and P.V
ffn              the two linear layers of a transformer block, forward: bias + ReLU, then bias
linear_backward  the two gradient products of a linear layer: dX = dY.W^T and dW = X^T.dY
conv             implicit-GEMM convolution with bias and ReLU, NHWC, channel counts multiples of 8
conv_any         the same for any channel counts (an RGB image), operands padded in a workspace
gemm_any         C = A.B for any extents and row pitches, operands padded in a workspace
"""
from __future__ import annotations

import math

import torch

import paper_2210_16691_amd as al

_DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
_CODE = {"f16": al.F16, "bf16": al.BF16, "f32": al.F32}
_SIZE = {"f16": 2, "bf16": 2, "f32": 4}


def listed():
    return [
        # the smallest call: a small product whose result is wanted in fp32 (launch latency)
        dict(name="gemm_256", kind="linear", M=256, N=256, K=256, dtype="f16", out="f32",
             transB=False, bias=False, relu=False),
        # the benchmark's headline product
        dict(name="gemm_2048", kind="linear", M=2048, N=2048, K=2048, dtype="f16", out="f16",
             transB=False, bias=False, relu=False),
        # a compute-bound square, the largest call
        dict(name="gemm_8192", kind="linear", M=8192, N=8192, K=8192, dtype="bf16", out="bf16",
             transB=False, bias=False, relu=False),
        # a classifier layer: small output, long reduction
        dict(name="fc_1024x64", kind="linear", M=1024, N=64, K=2048, dtype="f16", out="f16",
             transB=False, bias=False, relu=False),
        # a linear layer while decoding: a few tokens against a whole weight matrix, which is
        # stored as (out features, in features)
        dict(name="decode_16", kind="linear", M=16, N=3072, K=768, dtype="bf16", out="bf16",
             transB=True, bias=True, relu=False),
        # self-attention of 8 sequences x 12 heads, 512 tokens, head size 64 (prefill)
        dict(name="attention_512", kind="attention", batch=96, sq=512, sk=512, d=64, dtype="f16"),
        # the linear layers of a transformer block at 4096 tokens, forward
        dict(name="ffn_4096", kind="ffn", tokens=4096, d=768, hidden=3072, dtype="bf16"),
        # the gradients of the first of them, backward
        dict(name="linear_backward_4096", kind="linear_backward", tokens=4096, d=768, hidden=3072,
             dtype="bf16"),
        # 3x3 convolutions of an early and of a late residual stage, with the folded
        # normalisation's bias and the ReLU
        dict(name="conv_56", kind="conv", N=32, H=56, W=56, C=64, K=64, R=3, S=3, stride=1, pad=1,
             dtype="f16", krsc=False),
        dict(name="conv_14", kind="conv", N=32, H=14, W=14, C=256, K=256, R=3, S=3, stride=1, pad=1,
             dtype="f16", krsc=False),
        # the 7x7 stem of such a network on RGB images
        dict(name="conv_stem", kind="conv_any", N=32, H=224, W=224, C=3, K=64, R=7, S=7, stride=2,
             pad=3, dtype="f16"),
        # a product none of whose extents fits a tile or a 16-byte chunk
        dict(name="gemm_odd", kind="gemm_any", M=1021, N=1531, K=767, dtype="bf16"),
    ]


def _log(rng, lo, hi, mult=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(mult, int(round(v / mult)) * mult)


def draw(rng):
    while True:
        case = _draw(rng)
        w = work(case)
        if w["flops"] <= 4e11 and w["bytes"] <= 1.5e9:
            return case


def _draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "attention", "ffn", "linear_backward", "conv",
                       "conv", "conv_any", "gemm_any"])
    dtype = rng.choice(["f16", "bf16"])
    if kind == "linear":
        bias = rng.random() < 0.5
        return dict(kind=kind, M=_log(rng, 1, 8192), N=_log(rng, 64, 8192, 8), K=_log(rng, 64, 8192, 8),
                    dtype=dtype, out=rng.choice([dtype, dtype, dtype, "f32"]),
                    transB=rng.random() < 0.5, bias=bias, relu=bias and rng.random() < 0.5)
    if kind == "attention":
        return dict(kind=kind, batch=_log(rng, 4, 128), sq=_log(rng, 64, 2048), sk=_log(rng, 64, 2048, 8),
                    d=rng.choice([32, 64, 64, 80, 96, 128]), dtype=dtype)
    if kind in ("ffn", "linear_backward"):
        # tokens are the reduction axis of the weight gradient: a multiple of 8 there
        d = _log(rng, 256, 2048, 64)
        return dict(kind=kind, tokens=_log(rng, 128, 8192, 8 if kind == "linear_backward" else 1), d=d,
                    hidden=d * rng.choice([1, 2, 3, 4]), dtype=dtype)
    if kind == "conv":
        R = rng.choice([1, 3, 3, 3, 5])
        H = _log(rng, 7, 112)
        return dict(kind=kind, N=_log(rng, 1, 64), H=H, W=max(R, H + rng.choice([-1, 0, 0, 0, 2])),
                    C=_log(rng, 16, 512, rng.choice([8, 32, 64])), K=_log(rng, 16, 512, rng.choice([8, 32, 64])),
                    R=R, S=R, stride=rng.choice([1, 1, 1, 2]), pad=R // 2, dtype=dtype,
                    krsc=rng.random() < 0.25)
    if kind == "conv_any":
        R = rng.choice([3, 5, 7, 7])
        H = _log(rng, 28, 256)
        return dict(kind=kind, N=_log(rng, 1, 64), H=H, W=H + rng.choice([-3, 0, 0, 5]),
                    C=rng.choice([1, 3, 3, 3, 4, 6, 12]), K=rng.choice([16, 32, 48, 61, 64, 64, 96]),
                    R=R, S=R, stride=rng.choice([1, 2, 2, 4]), pad=R // 2, dtype=dtype)
    return dict(kind=kind, M=_log(rng, 16, 4096), N=_log(rng, 16, 4096), K=_log(rng, 16, 4096),
                dtype=dtype)


def _extent(case):
    p = (case["H"] + 2 * case["pad"] - case["R"]) // case["stride"] + 1
    q = (case["W"] + 2 * case["pad"] - case["S"]) // case["stride"] + 1
    return p, q


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    dt = _DT[case["dtype"]]

    def uniform(*shape):
        return torch.empty(shape, dtype=torch.float32, device=dev).uniform_(-1.0, 1.0, generator=g).to(dt)

    def normal(*shape, scale=1.0):
        return (torch.empty(shape, dtype=torch.float32, device=dev).normal_(generator=g) * scale).to(dt)

    def bias(n):
        return torch.empty(n, dtype=torch.float32, device=dev).normal_(generator=g) * 0.1

    def out(*shape, dtype=dt):
        return torch.empty(shape, dtype=dtype, device=dev)

    s = dict(case=case)
    kind = case["kind"]
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        s.update(A=uniform(M, K), B=uniform(N, K) if case["transB"] else uniform(K, N),
                 C=out(M, N, dtype=_DT[case["out"]]), bias=bias(N) if case["bias"] else None)
    elif kind == "attention":
        b, sq, sk, d = case["batch"], case["sq"], case["sk"], case["d"]
        logits = torch.empty((b, sq, sk), dtype=torch.float32, device=dev).normal_(generator=g)
        s.update(Q=normal(b, sq, d), Kt=normal(b, sk, d), V=normal(b, sk, d),
                 P=torch.softmax(logits, dim=-1).to(dt), scores=out(b, sq, sk), context=out(b, sq, d))
    elif kind == "ffn":
        t, d, h = case["tokens"], case["d"], case["hidden"]
        s.update(x=normal(t, d), w1=normal(d, h, scale=d ** -0.5), b1=bias(h),
                 w2=normal(h, d, scale=h ** -0.5), b2=bias(d), h=out(t, h), y=out(t, d))
    elif kind == "linear_backward":
        t, d, h = case["tokens"], case["d"], case["hidden"]
        s.update(x=normal(t, d), w=normal(d, h, scale=d ** -0.5), dy=normal(t, h, scale=t ** -0.5),
                 dx=out(t, d), dw=out(d, h))
    elif kind in ("conv", "conv_any"):
        p, q = _extent(case)
        scale = (case["R"] * case["S"] * case["C"]) ** -0.5
        wshape = (case["R"], case["S"], case["C"], case["K"])
        if case.get("krsc"):
            wshape = (case["K"], case["R"], case["S"], case["C"])
        s.update(x=normal(case["N"], case["H"], case["W"], case["C"]), w=normal(*wshape, scale=scale),
                 bias=bias(case["K"]), y=out(case["N"], p, q, case["K"]))
        if kind == "conv_any":
            n = al.alcop_conv2d_unaligned_workspace_bytes(
                case["N"], case["H"], case["W"], case["C"], case["K"], case["R"], case["S"],
                (case["stride"],) * 2, (case["pad"],) * 2, (1, 1), _CODE[case["dtype"]])
            s["workspace"] = torch.empty(n, dtype=torch.uint8, device=dev)
    else:
        M, N, K = case["M"], case["N"], case["K"]
        n = al.alcop_unaligned_workspace_bytes(1, M, N, K, _CODE[case["dtype"]])
        s.update(A=uniform(M, K), B=uniform(K, N), C=out(M, N), bias=bias(N),
                 workspace=torch.empty(n, dtype=torch.uint8, device=dev))
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "linear":
        if case["bias"]:
            return al.alcop_gemm_fused(s["A"], s["B"], s["C"], bias=s["bias"], act=int(case["relu"]),
                                       transB=case["transB"])
        return al.alcop_gemm(s["A"], s["B"], s["C"], transB=case["transB"])
    if kind == "attention":
        al.alcop_bmm_fused(s["Q"], s["Kt"], s["scores"], alpha=case["d"] ** -0.5, transB=True)
        al.alcop_bmm(s["P"], s["V"], s["context"])
        return s["scores"], s["context"]
    if kind == "ffn":
        al.alcop_gemm_fused(s["x"], s["w1"], s["h"], bias=s["b1"], act=1)
        al.alcop_gemm_fused(s["h"], s["w2"], s["y"], bias=s["b2"])
        return s["h"], s["y"]
    if kind == "linear_backward":
        al.alcop_gemm(s["dy"], s["w"], s["dx"], transB=True)
        al.alcop_gemm(s["x"], s["dy"], s["dw"], transA=True)
        return s["dx"], s["dw"]
    if kind == "conv":
        return al.alcop_conv2d_igemm_fused(s["x"], s["w"], s["y"], (case["stride"],) * 2,
                                           (case["pad"],) * 2, bias=s["bias"], act=1, krsc=case["krsc"])
    if kind == "conv_any":
        return al.alcop_conv2d_igemm_unaligned(s["x"], s["w"], s["y"], s["workspace"],
                                               (case["stride"],) * 2, (case["pad"],) * 2,
                                               bias=s["bias"], act=1)
    return al.alcop_bmm_unaligned(s["A"], s["B"], s["C"], s["workspace"], bias=s["bias"])


def work(case):
    kind = case["kind"]
    e = _SIZE[case["dtype"]]
    if kind in ("linear", "gemm_any"):
        M, N, K = case["M"], case["N"], case["K"]
        has_bias = case.get("bias", True)
        return dict(bytes=e * (M * K + K * N) + _SIZE[case.get("out", case["dtype"])] * M * N + (4 * N if has_bias else 0),
                    flops=2 * M * N * K)
    if kind == "attention":
        b, sq, sk, d = case["batch"], case["sq"], case["sk"], case["d"]
        return dict(bytes=e * b * (sq * d + sk * d + sq * sk + sq * sk + sk * d + sq * d),
                    flops=4 * b * sq * sk * d)
    if kind == "ffn":
        t, d, h = case["tokens"], case["d"], case["hidden"]
        # the hidden activations are an output of the first layer; the second reads them again
        return dict(bytes=e * (t * d + d * h + t * h + t * h + h * d + t * d) + 4 * (d + h), flops=4 * t * d * h)
    if kind == "linear_backward":
        t, d, h = case["tokens"], case["d"], case["hidden"]
        return dict(bytes=e * (t * h + d * h + t * d + t * d + d * h), flops=4 * t * d * h)
    p, q = _extent(case)
    outs = case["N"] * p * q * case["K"]
    k = case["R"] * case["S"] * case["C"]
    return dict(bytes=e * (case["N"] * case["H"] * case["W"] * case["C"] + k * case["K"] + outs) + 4 * case["K"],
                flops=2 * outs * k)


def tolerance(case):
    # Against the same products in fp64 (fp32 accumulation here): about 2.1e-4 for fp16 and 1.7e-3
    # for bf16 results, which is the rounding of the output; for fp32 results 1.0e-7 with K = 256
    # and 5.7e-7 with K = 8192.  Four times that.
    if case.get("out") == "f32":
        return dict(rel=4e-7 if case["K"] <= 256 else 2.3e-6)
    return dict(rel=8e-4) if case["dtype"] == "f16" else dict(rel=7e-3)
