"""Performance cases: the work that programs have this library do, through its
public entry points, over the sizes, types and layouts they use.

Kinds of case (the "kind" of a case):

* ``matmul``: one product of two matrices, A row-major and B row-major or (a
  linear layer's weight, stored output-major) column-major;
* ``train``: the differentiable product with both gradients;
* ``fp8``: an FP8 linear layer, activations quantised on every call, weights
  quantised once (or, ``both``, both operands on every call);
* ``grouped``: problems of different heights in one launch (routed tokens);
* ``batched``: equal problems in one launch;
* ``conv``: a channels-last convolution.
"""
import math

import torch

from paper_2212_08964_amd import autograd, skgemm

DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32, "f64": torch.float64}
BYTES = {"bf16": 2, "f16": 2, "f32": 4, "f64": 8}


def listed():
    return [
        # the smallest product of the FP32 path: 9 tiles of 128 x 128 on 256 CUs, a call bound by latency and its split
        {"name": "f32_384", "kind": "matmul", "dtype": "f32", "m": 384, "n": 384, "k": 1024, "b_col": False},
        # a small layer: one tile per CU and less, where launch, fill and drain of the pipeline count
        {"name": "f16_1024", "kind": "matmul", "dtype": "f16", "m": 1024, "n": 1024, "k": 1024, "b_col": False},
        # the large square product: the matrix cores' rate
        {"name": "bf16_8192", "kind": "matmul", "dtype": "bf16", "m": 8192, "n": 8192, "k": 8192, "b_col": False},
        # a mid-size product with every dimension odd or unaligned, from the ragged half of the shape sweep
        {"name": "bf16_ragged", "kind": "matmul", "dtype": "bf16", "m": 4427, "n": 2519, "k": 3013, "b_col": False},
        # a linear layer over a short prompt: the weight streams once
        {"name": "bf16_prompt_128", "kind": "matmul", "dtype": "bf16", "m": 128, "n": 8192, "k": 8192, "b_col": True},
        # the same layer in decoding: a few rows, bound by the weight's bytes
        {"name": "bf16_decode_16", "kind": "matmul", "dtype": "bf16", "m": 16, "n": 8192, "k": 8192, "b_col": True},
        # double precision at a size no tile divides
        {"name": "f64_mid", "kind": "matmul", "dtype": "f64", "m": 3000, "n": 2000, "k": 1500, "b_col": False},
        # a training step's three products
        {"name": "bf16_train", "kind": "train", "dtype": "bf16", "m": 2048, "n": 2048, "k": 8192},
        # FP8 inference: activations quantised on the way in
        {"name": "fp8_linear", "kind": "fp8", "dtype": "bf16", "m": 4096, "n": 8192, "k": 8192, "both": False},
        # routed tokens: 64 problems whose heights follow Zipf's law
        {"name": "bf16_grouped", "kind": "grouped", "dtype": "bf16", "g": 64, "n": 4096, "k": 2048, "shape_seed": 0},
        # many equal products with a long reduction
        {"name": "bf16_batched", "kind": "batched", "dtype": "bf16", "batch": 32, "m": 128, "n": 256, "k": 2048},
        # a 3 x 3 layer of a ResNet-50 at batch 32
        {"name": "bf16_conv", "kind": "conv", "dtype": "bf16", "batch": 32, "h": 28, "w": 28, "c": 128, "f": 128,
         "r": 3, "pad": 1, "stride": 1},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng, lo, hi):
    """A dimension spread over the logarithm of its range: half of them multiples of 128 (64 below 256), half as drawn."""
    v = _log(rng, lo, hi)
    if rng.random() < 0.5:
        q = 128 if v >= 256 else 64
        v = max(q, round(v / q) * q)
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["matmul"] * 5 + ["decode"] * 2 + ["train", "fp8", "grouped", "batched", "conv"])
    if kind == "matmul":
        dtype = rng.choice(["bf16", "bf16", "f16", "f32", "f64"])
        hi = {"f32": 4096, "f64": 3072}.get(dtype, 8192)
        most = {"f32": 7e10, "f64": 3.5e10}.get(dtype, 1.1e12)      # what the type's rate does in the largest listed case's time
        while True:
            m, n, k = (_dim(rng, 128, hi) for _ in range(3))
            if 2.0 * m * n * k <= most:
                break
        return {"kind": "matmul", "dtype": dtype, "m": m, "n": n, "k": k, "b_col": rng.random() < 0.5}
    if kind == "decode":
        return {"kind": "matmul", "dtype": rng.choice(["bf16", "f16"]), "m": _log(rng, 1, 160),
                "n": _dim(rng, 1024, 16384), "k": _dim(rng, 1024, 8192), "b_col": rng.random() < 0.75}
    if kind == "train":
        return {"kind": "train", "dtype": rng.choice(["bf16", "f16"]), "m": _dim(rng, 256, 4096),
                "n": _dim(rng, 512, 4096), "k": _dim(rng, 512, 8192)}
    if kind == "fp8":
        return {"kind": "fp8", "dtype": rng.choice(["bf16", "bf16", "f32"]), "m": _dim(rng, 128, 8192),
                "n": _dim(rng, 1024, 8192), "k": _dim(rng, 1024, 8192), "both": rng.random() < 0.3}
    if kind == "grouped":
        return {"kind": "grouped", "dtype": rng.choice(["bf16", "f16"]), "g": rng.randint(8, 64),
                "n": _dim(rng, 512, 4096), "k": _dim(rng, 512, 2048), "shape_seed": rng.randint(0, 1000)}
    if kind == "batched":
        return {"kind": "batched", "dtype": rng.choice(["bf16", "f16"]), "batch": _log(rng, 4, 64),
                "m": _dim(rng, 64, 1024), "n": _dim(rng, 64, 1024), "k": _dim(rng, 128, 2048)}
    h = rng.choice([7, 14, 28, 56])
    c = rng.choice([64, 128, 256]) if h > 14 else rng.choice([256, 512])
    r = rng.choice([1, 3])
    return {"kind": "conv", "dtype": rng.choice(["bf16", "f16"]), "batch": _log(rng, 4, 32), "h": h, "w": h, "c": c,
            "f": rng.choice([64, 128, 256]) if h > 14 else rng.choice([256, 512]), "r": r, "pad": r // 2,
            "stride": rng.choice([1, 1, 2])}


def heights(case):
    """Rows of each problem of a grouped case: Zipf(1.2) on [16, 4096]."""
    import numpy as np
    m = np.arange(16, 4097, dtype=np.float64)
    cdf = np.cumsum(m ** -1.2)
    u = np.random.default_rng(case["shape_seed"]).random(case["g"])
    return [int(m[i]) for i in np.searchsorted(cdf / cdf[-1], u)]


def _inputs(case, seed):
    """The case's floating inputs on the GPU, N(0, 1), and weights scaled by the square root of the reduction's length."""
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)

    def normal(shape, scale=1.0, dtype=DTYPES[case["dtype"]]):
        x = torch.randn(shape, generator=g, device="cuda:0", dtype=torch.float64 if dtype == torch.float64 else torch.float32)
        return (x * scale).to(dtype)

    kind = case["kind"]
    if kind == "conv":
        taps = case["r"] * case["r"] * case["c"]
        return (normal((case["batch"], case["h"], case["w"], case["c"])),
                normal((case["f"], case["r"], case["r"], case["c"]), taps ** -0.5))
    n, k = case["n"], case["k"]
    if kind == "grouped":
        ms = heights(case)
        return [normal((m, k)) for m in ms], [normal((k, n), k ** -0.5) for _ in ms]
    if kind == "batched":
        return normal((case["batch"], case["m"], k)), normal((case["batch"], k, n), k ** -0.5)
    a = normal((case["m"], k))
    if kind == "fp8" or (kind == "matmul" and case["b_col"]):
        b = normal((n, k), k ** -0.5).t()
    else:
        b = normal((k, n), k ** -0.5)
    if kind == "train":
        return a, b, normal((case["m"], n))
    return a, b


def prepare(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "train":
        x = (x[0].requires_grad_(), x[1].requires_grad_(), x[2])
    if case["kind"] == "fp8" and not case["both"]:
        x = (x[0],) + tuple(skgemm.quantize_e4m3(x[1], layout="col"))
    return {"case": case, "x": x}


def run(state):
    case, x = state["case"], state["x"]
    kind = case["kind"]
    if kind == "matmul":
        return skgemm.matmul(x[0], x[1])
    if kind == "train":
        c = autograd.skgemm_matmul(x[0], x[1])
        da, db = torch.autograd.grad(c, (x[0], x[1]), x[2])
        return {"c": c.detach(), "da": da, "db": db}
    if kind == "fp8":
        if case["both"]:
            c, (qa, sa), (qb, sb) = skgemm.matmul_fp8(x[0], x[1], out_dtype=torch.bfloat16)
            return {"c": c, "qa": qa, "sa": sa, "qb": qb, "sb": sb}
        qa, sa = skgemm.quantize_e4m3(x[0])
        return {"c": skgemm.matmul(qa, x[1], out_dtype=torch.bfloat16, scale_a=sa, scale_b=x[2]), "qa": qa, "sa": sa}
    if kind == "grouped":
        return skgemm.grouped_matmul(x[0], x[1])[0]
    if kind == "batched":
        return skgemm.batched_matmul(x[0], x[1])
    p = case["pad"]
    return skgemm.conv2d(x[0], x[1], padding=(p, p), stride=(case["stride"],) * 2)


def _out_size(case):
    return (case["h"] + 2 * case["pad"] - case["r"]) // case["stride"] + 1


def work(case):
    kind, e = case["kind"], BYTES[case["dtype"]]
    if kind == "conv":
        out = case["batch"] * _out_size(case) ** 2 * case["f"]
        taps = case["r"] * case["r"] * case["c"]
        return {"bytes": e * (case["batch"] * case["h"] * case["w"] * case["c"] + case["f"] * taps + out),
                "flops": 2 * out * taps}
    n, k = case["n"], case["k"]
    if kind == "grouped":
        ms = heights(case)
        return {"bytes": e * (sum(ms) * (n + k) + len(ms) * n * k), "flops": 2 * sum(ms) * n * k}
    m, times = case["m"], case.get("batch", 1)
    one = m * k + k * n + m * n
    if kind == "train":         # A, B and dC in, C, dA and dB out
        return {"bytes": e * 2 * one, "flops": 6 * m * n * k}
    if kind == "fp8":           # inputs, the quantised copies, and the 16-bit result
        b = k * n * (e + 1) if case["both"] else k * n
        return {"bytes": m * k * (e + 1) + b + 2 * m * n, "flops": 2 * m * n * k}
    return {"bytes": times * e * one, "flops": times * 2 * m * n * k}


def _codes(x):
    """E4M3 codes of x under the per-tensor scale absmax / 448, as float64 values, and the scale."""
    s = (x.double().abs().max() / 448.0).float()
    q = (x.float() / s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return q.float().double(), s.double().reshape(1)


def exact(case, seed):
    x, kind = _inputs(case, seed), case["kind"]
    if kind == "matmul":
        return x[0].double() @ x[1].double()
    if kind == "train":
        a, b, dc = (t.double() for t in x)
        return {"c": a @ b, "da": dc @ b.t(), "db": a.t() @ dc}
    if kind == "fp8":
        (qa, sa), (qb, sb) = _codes(x[0]), _codes(x[1])
        out = {"c": (qa @ qb) * (sa * sb), "qa": qa, "sa": sa}
        if case["both"]:
            out.update(qb=qb, sb=sb)
        return out
    if kind == "grouped":
        return [a.double() @ b.double() for a, b in zip(*x)]
    if kind == "batched":
        return torch.stack([a.double() @ b.double() for a, b in zip(*x)])
    p, st, r, o = case["pad"], case["stride"], case["r"], _out_size(case)
    xp = torch.nn.functional.pad(x[0].double(), (0, 0, p, p, p, p))
    y = 0
    for i in range(r):
        for j in range(r):
            y = y + xp[:, i:i + (o - 1) * st + 1:st, j:j + (o - 1) * st + 1:st, :] @ x[1][:, i, j, :].double().t()
    return y
