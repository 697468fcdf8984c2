"""Workloads of the library, one dict each, that a program can prepare and run through the public entry points.

Five families: plain products (gemm / addmm / bmm), convolutions, attention, row-wise kernels.  Sizes are those of this
repository's benchmark configurations and of the paper's task list, plus the calls that such programs make around them:
a decoding step's skinny product and one-query attention, ragged sizes, a strided convolution."""
import math

import torch

import paper_2507_11978_amd as nt

_DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest call: the benchmark's tiny product on the tile its configuration names; latency is all there is to it
        dict(name="mm_256_tile64", op="mm", M=256, N=256, K=256, dtype="f16", out="f16", bt=False, tile64=True, dist="uniform"),
        # one linear layer of a decoding step over 16 sequences: weights stored [out, in], read once per call
        dict(name="mm_decode", op="mm", M=16, N=4096, K=4096, dtype="f16", out="f16", bt=True, tile64=False, dist="normal"),
        # no dimension a multiple of anything: the benchmark's masked-edge product, fp32 result
        dict(name="mm_ragged", op="mm", M=3001, N=5003, K=1999, dtype="bf16", out="f32", bt=False, tile64=False, dist="uniform"),
        # the headline: the largest square product
        dict(name="mm_8192", op="mm", M=8192, N=8192, K=8192, dtype="f16", out="f16", bt=False, tile64=False, dist="normal"),
        # a linear layer of an MLP over a full batch: bias and activation fused into the product
        dict(name="addmm_gelu_4096", op="addmm", M=4096, N=4096, K=4096, dtype="f16", out="f16", bt=False, bias="row", act="gelu_tanh"),
        # batched product, short reduction: attention-like matmuls written as bmm
        dict(name="bmm_32x2048", op="bmm", B=32, M=2048, N=2048, K=512, dtype="f16", out="f16"),
        # a 3 x 3 layer of an image network over a training batch
        dict(name="conv_56", op="conv", N=32, C=256, H=56, W=56, F=256, R=3, stride=1, pad=1, dtype="f16"),
        # the paper's conv2d task: few positions, a long reduction
        dict(name="conv_14", op="conv", N=4, C=512, H=14, W=14, F=512, R=3, stride=1, pad=0, dtype="f16"),
        # a downsampling layer: stride 2
        dict(name="conv_stride2", op="conv", N=32, C=128, H=56, W=56, F=256, R=3, stride=2, pad=1, dtype="f16"),
        # attention over a whole prompt: the paper's sdpa task
        dict(name="sdpa_prefill", op="sdpa", B=4, H=48, Sq=1024, Sk=1024, dtype="f16"),
        # attention of one decoding step: a single query per head against a cache of odd length
        dict(name="sdpa_decode", op="sdpa", B=4, H=48, Sq=1, Sk=2047, dtype="bf16"),
        # row-wise kernel on rows of odd length (scores of a ragged problem)
        dict(name="softmax_ragged", op="softmax", rows=3001, cols=5003, dtype="bf16"),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _dim(rng, lo, hi):
    """A size of [lo, hi]: as it falls, a multiple of 8, or a multiple of 64."""
    v, unit = _log(rng, lo, hi), rng.choice([1, 8, 64])
    return min(hi, max(lo, v // unit * unit))


def draw(rng):
    dtype = rng.choice(["f16", "bf16"])
    op = rng.choice(["small", "decode", "large", "addmm", "bmm", "conv", "conv", "conv2", "sdpa", "sdpa1", "rows"])
    if op == "small":
        tile64 = rng.random() < 0.5
        return dict(op="mm", M=_dim(rng, 32, 512), N=_dim(rng, 32, 512), K=_dim(rng, 32, 1024), dtype=dtype, out=rng.choice([dtype, "f32"]),
                    bt=rng.random() < 0.5, tile64=tile64, dist="normal")
    if op == "decode":
        return dict(op="mm", M=_log(rng, 1, 64), N=_dim(rng, 1024, 8192), K=_dim(rng, 1024, 8192), dtype=dtype, out=dtype,
                    bt=rng.random() < 0.5, tile64=False, dist="normal")
    if op == "large":
        return dict(op="mm", M=_dim(rng, 512, 8192), N=_dim(rng, 512, 8192), K=_dim(rng, 512, 8192), dtype=dtype, out=rng.choice([dtype, "f32"]),
                    bt=rng.random() < 0.5, tile64=False, dist="normal")
    if op == "addmm":
        return dict(op="addmm", M=_dim(rng, 256, 4096), N=_dim(rng, 512, 4096), K=_dim(rng, 512, 4096), dtype=dtype, out=dtype,
                    bt=rng.random() < 0.5, bias=rng.choice(["row", "full"]), act=rng.choice(["none", "relu", "silu", "gelu_tanh"]))
    if op == "bmm":
        return dict(op="bmm", B=_log(rng, 2, 32), M=_dim(rng, 128, 2048), N=_dim(rng, 128, 2048), K=_dim(rng, 64, 2048), dtype=dtype, out=dtype)
    if op in ("conv", "conv2"):
        stride = 2 if op == "conv2" else 1
        H = rng.choice([14, 27, 28, 56]) if stride == 2 else rng.choice([7, 13, 14, 28, 56])
        R = rng.choice([1, 3, 3, 5])
        return dict(op="conv", N=_log(rng, 1, 32), C=32 * _log(rng, 2, 16), H=H, W=H, F=_dim(rng, 64, 512), R=R, stride=stride, pad=R // 2, dtype=dtype)
    if op == "sdpa":
        return dict(op="sdpa", B=_log(rng, 1, 4), H=_log(rng, 8, 48), Sq=_dim(rng, 64, 2048), Sk=_dim(rng, 64, 2048), dtype=dtype)
    if op == "sdpa1":
        return dict(op="sdpa", B=_log(rng, 1, 16), H=_log(rng, 8, 48), Sq=1, Sk=_log(rng, 128, 4096), dtype=dtype)
    return dict(op=rng.choice(["softmax", "rms_norm"]), rows=_log(rng, 1, 8192), cols=_dim(rng, 128, 8192), dtype=dtype)


def _out_size(c):
    return (c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1


def _inputs(c, seed):
    """The operands, made on the GPU from the seed: fp32 draws rounded once to the storage type."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + 17)
    dt = _DT[c["dtype"]]

    def normal(shape, scale):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale).to(dt)

    def uniform(shape):
        return (torch.rand(shape, generator=g, device="cuda", dtype=torch.float32) * 2 - 1).to(dt)

    op = c["op"]
    if op in ("mm", "addmm"):
        M, N, K = c["M"], c["N"], c["K"]
        shape_b = (N, K) if c["bt"] else (K, N)
        if c.get("dist") == "uniform":
            a, b = uniform((M, K)), uniform(shape_b)
        else:
            a, b = normal((M, K), K ** -0.25), normal(shape_b, K ** -0.25)      # entries of the product of order one
        s = dict(a=a, b=b.t() if c["bt"] else b)
        if op == "addmm":
            s["bias"] = torch.randn((N,) if c["bias"] == "row" else (M, N), generator=g, device="cuda", dtype=torch.float32).to(_DT[c["out"]])
        return s
    if op == "bmm":
        B, M, N, K = c["B"], c["M"], c["N"], c["K"]
        return dict(a=normal((B, M, K), K ** -0.25), b=normal((B, K, N), K ** -0.25))
    if op == "conv":
        fan = c["C"] * c["R"] * c["R"]
        return dict(x=normal((c["N"], c["C"], c["H"], c["W"]), 1.0), w=normal((c["F"], c["C"], c["R"], c["R"]), fan ** -0.5))
    if op == "sdpa":
        return dict(q=normal((c["B"], c["H"], c["Sq"], 64), 1.0), k=normal((c["B"], c["H"], c["Sk"], 64), 1.0), v=normal((c["B"], c["H"], c["Sk"], 64), 1.0))
    return dict(x=normal((c["rows"], c["cols"]), 2.0))


def prepare(case, seed):
    s = _inputs(case, seed)
    op = case["op"]
    if op in ("mm", "addmm"):
        shape, dt = (case["M"], case["N"]), _DT[case["out"]]
    elif op == "bmm":
        shape, dt = (case["B"], case["M"], case["N"]), _DT[case["out"]]
    elif op == "conv":
        shape, dt = (case["N"], case["F"], *_out_size(case)), _DT[case["dtype"]]
    elif op == "sdpa":
        shape, dt = s["q"].shape, _DT[case["dtype"]]
    else:
        shape, dt = s["x"].shape, _DT[case["dtype"]]
    s["out"] = torch.empty(shape, dtype=dt, device="cuda")
    s["case"] = case
    return s


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "mm":
        return nt.gemm(s["a"], s["b"], s["out"], tile=(64, 64, 32) if c["tile64"] else None)
    if op == "addmm":
        return nt.addmm(s["bias"], s["a"], s["b"], s["out"], act=c["act"])
    if op == "bmm":
        return nt.bmm(s["a"], s["b"], s["out"])
    if op == "conv":
        return nt.conv2d_implicit(s["x"], s["w"], s["out"], (c["stride"], c["stride"]), (c["pad"], c["pad"]))
    if op == "sdpa":
        return nt.sdpa(s["q"], s["k"], s["v"], s["out"])
    if op == "softmax":
        return nt.softmax(s["x"], s["out"])
    return nt.rms_norm(s["x"], s["out"], eps=1e-6)


def work(c):
    op = c["op"]
    if op in ("mm", "addmm"):
        M, N, K, osz = c["M"], c["N"], c["K"], 4 if c["out"] == "f32" else 2
        extra = 0 if op == "mm" else osz * (N if c["bias"] == "row" else M * N)
        return {"bytes": 2 * (M * K + K * N) + osz * M * N + extra, "flops": 2 * M * N * K}
    if op == "bmm":
        B, M, N, K = c["B"], c["M"], c["N"], c["K"]
        return {"bytes": 2 * B * (M * K + K * N + M * N), "flops": 2 * B * M * N * K}
    if op == "conv":
        P, Q = _out_size(c)
        rr = c["C"] * c["R"] * c["R"]
        return {"bytes": 2 * (c["N"] * c["C"] * c["H"] * c["W"] + c["F"] * rr + c["N"] * c["F"] * P * Q), "flops": 2 * c["N"] * P * Q * c["F"] * rr}
    if op == "sdpa":
        bh = c["B"] * c["H"]
        return {"bytes": 2 * bh * 64 * (2 * c["Sq"] + 2 * c["Sk"]), "flops": 4 * bh * c["Sq"] * c["Sk"] * 64}
    n = c["rows"] * c["cols"]
    return {"bytes": 4 * n, "flops": (5 if op == "softmax" else 3) * n}


def tolerance(c):
    """Four times the relative error against 64 bits of one rounding to the result's type (2.1e-4 fp16, 1.7e-3 bf16;
    attention, which also rounds its weights to the type, 3e-4 / 2.5e-3), one unit in the last place twice for the largest."""
    out = c.get("out", c["dtype"])
    if out == "f32":
        return {"rel": 1e-5}
    if c["op"] == "sdpa":
        return {"rel": 1.2e-3, "max": 1e-2} if out == "f16" else {"rel": 1e-2, "max": 8e-2}
    return {"rel": 8e-4, "max": 4e-3} if out == "f16" else {"rel": 6.6e-3, "max": 3.2e-2}


def exact(c, seed):
    s = {k: v.double() for k, v in _inputs(c, seed).items()}
    op = c["op"]
    if op == "mm":
        return s["a"] @ s["b"]
    if op == "addmm":
        y = s["a"] @ s["b"] + s["bias"]
        if c["act"] == "relu":
            return torch.clamp(y, min=0)
        if c["act"] == "silu":
            return y * torch.sigmoid(y)
        if c["act"] == "gelu_tanh":
            return 0.5 * y * (1 + torch.tanh(math.sqrt(2 / math.pi) * (y + 0.044715 * y ** 3)))
        return y
    if op == "bmm":
        return torch.bmm(s["a"], s["b"])
    if op == "conv":
        P, Q = _out_size(c)
        w = s["w"].reshape(c["F"], -1)
        cols = (torch.nn.functional.unfold(x[None], (c["R"], c["R"]), padding=c["pad"], stride=c["stride"])[0] for x in s["x"])
        return torch.stack([(w @ u).reshape(c["F"], P, Q) for u in cols])
    if op == "sdpa":
        rows = []
        for q, k, v in zip(s["q"], s["k"], s["v"]):
            p = torch.softmax(torch.bmm(q, k.transpose(1, 2).contiguous()) * 0.125, dim=-1)
            rows.append(torch.bmm(p, v))
        return torch.stack(rows)
    if op == "softmax":
        return torch.softmax(s["x"], dim=-1)
    return s["x"] / torch.sqrt((s["x"] ** 2).mean(dim=-1, keepdim=True) + 1e-6)
