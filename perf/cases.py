"""The work that a user has this library do, as cases that can be timed and compared: plain calls through the Python
binding of the C ABI, with no configuration named and nothing tuned beforehand.

A case is one of five kinds:

  gemm       one fused GEMM (hidet_gemm): any extents, transposes, bias / residual / ReLU, 16-bit or fp32
  mlp        the two fused GEMMs of a transformer MLP: up-projection + bias + ReLU, down-projection + bias + residual
  attention  scores = alpha Q.K^T, row softmax, context = P.V, for batch x heads independent entries (three calls)
  conv       one fused convolution, NCHW (bias + ReLU, residual), from OIHW weights or from repacked ones
  rows       one row softmax or row reduction

Inputs have the distributions of paper_2210_09603_amd/workloads.py and are drawn on the GPU from the seed.  Buffers for
the results, the epilogue descriptors and repacked weights are what a user's program keeps beside its weights, so they
belong to the state.
"""
import math

import torch

from paper_2210_09603_amd import binding as hb

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def _gemm(name, dtype, M, N, K, ta=False, tb=False, bias="col", residual=False, relu=True):
    return dict(name=name, kind="gemm", dtype=dtype, M=M, N=N, K=K, ta=ta, tb=tb, bias=bias, residual=residual, relu=relu)


def _mlp(name, dtype, tokens, d, ffn):
    return dict(name=name, kind="mlp", dtype=dtype, tokens=tokens, d=d, ffn=ffn)


def _attention(name, dtype, bh, seq, d=64):
    return dict(name=name, kind="attention", dtype=dtype, bh=bh, seq=seq, d=d)


def _conv(name, dtype, batch, ic, hw, oc, k, stride, residual=False, packed=False):
    return dict(name=name, kind="conv", dtype=dtype, batch=batch, ic=ic, hw=hw, oc=oc, k=k, stride=stride, pad=k // 2,
                residual=residual, packed=packed)


def _rows(name, dtype, op, rows, cols):
    return dict(name=name, kind="rows", dtype=dtype, op=op, rows=rows, cols=cols)


def listed():
    return [
        # the smallest fp32 product: launch and one latency chain
        _gemm("gemm_f32_256", "f32", 256, 256, 256),
        # the headline: a large square product, one that fills the matrix cores
        _gemm("gemm_f16_4096", "f16", 4096, 4096, 4096),
        # a prime extent: no row is aligned to more than its elements, no tile divides it
        _gemm("gemm_f16_2039", "f16", 2039, 2039, 2039),
        # transformer MLP of one layer: a decoding step of a few sequences, one short sequence, a full batch
        _mlp("mlp_f16_8_tokens", "f16", 8, 768, 3072),
        _mlp("mlp_f16_128_tokens", "f16", 128, 768, 3072),
        _mlp("mlp_bf16_4096_tokens", "bf16", 4096, 768, 3072),
        # attention of one sequence of 128 with 12 heads, and of a batch of 16 sequences of 512
        _attention("attention_f16_12x128", "f16", 12, 128),
        _attention("attention_f16_192x512", "f16", 192, 512),
        # bottleneck convolutions: one image (latency), a batch (throughput), and a 1x1 layer with 49 pixels an image
        _conv("conv3x3_f16_1x128x28", "f16", 1, 128, 28, 128, 3, 1),
        _conv("conv3x3_bf16_64x256x14", "bf16", 64, 256, 14, 256, 3, 1),
        _conv("conv1x1_f16_64x512x7", "f16", 64, 512, 7, 2048, 1, 1, residual=True),
        # next-token distribution over a vocabulary of 50257: long rows that no 16-byte access divides
        _rows("softmax_bf16_1024x50257", "bf16", "softmax", 1024, 50257),
    ]


def _spread(rng, lo, hi):
    """A whole number spread over [lo, hi] by its logarithm; half of them rounded to a multiple of 8 or 64, as most
    extents in use are, the rest left as they fall."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    step = rng.choice((1, 1, 8, 64))
    if v >= 2 * step:
        v = v // step * step
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(("gemm", "gemm", "mlp", "attention", "conv", "conv", "rows"))
    dtype = rng.choice(("f16", "bf16"))
    if kind == "gemm":
        if rng.random() < 0.3:
            dtype = "f32"
        top = 1536 if dtype == "f32" else 4096  # (an fp32 product costs sixteen times as much)
        c = _gemm("", dtype, _spread(rng, 16, top), _spread(rng, 16, top), _spread(rng, 16, top), ta=rng.random() < 0.2,
                  tb=rng.random() < 0.4, bias=rng.choice(("none", "col", "col", "row")), residual=rng.random() < 0.3,
                  relu=rng.random() < 0.5)
    elif kind == "mlp":
        d = rng.choice((512, 768, 1024))
        c = _mlp("", dtype, _spread(rng, 1, 4096), d, 4 * d)
    elif kind == "attention":
        seq = _spread(rng, 16, 512)
        c = _attention("", dtype, _spread(rng, 1, 192), seq, d=rng.choice((32, 64, 64, 128)))
    elif kind == "conv":
        ic, hw = rng.choice(((64, 56), (128, 28), (256, 14), (512, 7)))
        k = rng.choice((1, 3, 3, 5))
        stride = rng.choice((1, 1, 2))
        hw += rng.choice((0, 0, 0, -1, 1, 3))
        oc = rng.choice((ic, ic, 2 * ic, 4 * ic)) if k == 1 else ic
        c = _conv("", dtype, _spread(rng, 1, 64), ic, hw, oc, k, stride, residual=rng.random() < 0.3,
                  packed=k > 1 and rng.random() < 0.25)
    else:
        if rng.random() < 0.3:
            dtype = "f32"
        cols = _spread(rng, 16, 65536)
        rows = _spread(rng, 1, min(65536, 50_000_000 // cols))
        c = _rows("", dtype, rng.choice(("softmax", "softmax", "sum", "mean", "max")), rows, cols)
    del c["name"]
    return c


class _Draw:
    """Seeded inputs on the GPU."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))
        self.dtype = DTYPES[dtype]

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device="cuda").mul_(2).sub_(1).to(self.dtype)

    def normal(self, *shape, std=1.0):
        return torch.randn(shape, generator=self.g, device="cuda").mul_(std).to(self.dtype)

    def empty(self, *shape):
        return torch.empty(shape, dtype=self.dtype, device="cuda")


def prepare(case, seed):
    s = dict(case)
    r = _Draw(seed, case["dtype"])
    kind = case["kind"]
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        s["A"] = r.uniform(K, M) if case["ta"] else r.uniform(M, K)
        s["B"] = r.uniform(N, K) if case["tb"] else r.uniform(K, N)
        s["C"] = r.empty(M, N)
        axis = {"none": hb.HIDET_BIAS_NONE, "col": hb.HIDET_BIAS_PER_COL, "row": hb.HIDET_BIAS_PER_ROW}[case["bias"]]
        bias = None if case["bias"] == "none" else r.uniform(N if case["bias"] == "col" else M)
        s["epilogue"] = hb.make_epilogue(bias=bias, bias_axis=axis, residual=r.uniform(M, N) if case["residual"] else None,
                                         relu=case["relu"])
    elif kind == "mlp":
        t, d, f = case["tokens"], case["d"], case["ffn"]
        s["x"] = r.normal(t, d)
        s["w1"], s["w2"] = r.normal(d, f, std=0.02), r.normal(f, d, std=0.02)
        s["h"], s["y"] = r.empty(t, f), r.empty(t, d)
        s["up"] = hb.make_epilogue(bias=r.normal(f, std=0.02), bias_axis=hb.HIDET_BIAS_PER_COL, relu=True)
        s["down"] = hb.make_epilogue(bias=r.normal(d, std=0.02), bias_axis=hb.HIDET_BIAS_PER_COL, residual=s["x"])
    elif kind == "attention":
        b, n, d = case["bh"], case["seq"], case["d"]
        s["q"], s["k"], s["v"] = r.normal(b, n, d), r.normal(b, n, d), r.normal(b, n, d)
        s["p"], s["o"] = r.empty(b, n, n), r.empty(b, n, d)
        s["scale"] = hb.make_epilogue(alpha=1.0 / math.sqrt(d))
    elif kind == "conv":
        b, ic, hw, oc, k = case["batch"], case["ic"], case["hw"], case["oc"], case["k"]
        s["x"] = r.normal(b, ic, hw, hw)
        w = r.normal(oc, ic, k, k, std=math.sqrt(2.0 / (ic * k * k)))
        s["w"] = hb.hidet_conv2d_pack_weights(w) if case["packed"] else w
        s["strides"], s["pads"] = (case["stride"],) * 2, (case["pad"],) * 2
        s["y"] = r.empty(*hb.conv_out_shape(s["x"].shape, w.shape, s["strides"], s["pads"]))
        residual = r.normal(*s["y"].shape) if case["residual"] else None
        s["epilogue"] = hb.make_epilogue(bias=r.normal(oc, std=0.1), bias_axis=hb.HIDET_BIAS_PER_ROW, residual=residual,
                                         relu=True)
    else:
        s["x"] = r.normal(case["rows"], case["cols"], std=3.0 if case["op"] == "softmax" else 1.0)
        if case["op"] != "softmax":
            s["x"] += 0.25
        s["y"] = torch.empty_like(s["x"]) if case["op"] == "softmax" else r.empty(case["rows"])
    return s


_REDUCE = {"sum": hb.HIDET_REDUCE_SUM, "mean": hb.HIDET_REDUCE_MEAN, "max": hb.HIDET_REDUCE_MAX}


def run(s):
    kind = s["kind"]
    if kind == "gemm":
        hb.hidet_gemm(s["A"], s["B"], s["C"], transA=s["ta"], transB=s["tb"], epilogue=s["epilogue"])
        return s["C"]
    if kind == "mlp":
        hb.hidet_gemm(s["x"], s["w1"], s["h"], epilogue=s["up"])
        hb.hidet_gemm(s["h"], s["w2"], s["y"], epilogue=s["down"])
        return s["h"], s["y"]
    if kind == "attention":
        hb.hidet_batched_gemm(s["q"], s["k"], s["p"], transB=True, epilogue=s["scale"])
        hb.hidet_softmax_rows(s["p"], s["p"])
        hb.hidet_batched_gemm(s["p"], s["v"], s["o"])
        return s["p"], s["o"]
    if kind == "conv":
        conv = hb.hidet_conv2d_implicit_gemm_packed if s["packed"] else hb.hidet_conv2d_implicit_gemm
        conv(s["x"], s["w"], s["y"], stride=s["strides"], pad=s["pads"], epilogue=s["epilogue"])
        return s["y"]
    if s["op"] == "softmax":
        hb.hidet_softmax_rows(s["x"], s["y"])
    else:
        hb.hidet_reduce_rows(s["x"], s["y"], op=_REDUCE[s["op"]])
    return s["y"]


def work(case):
    e, kind = BYTES[case["dtype"]], case["kind"]
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        bias = {"none": 0, "col": N, "row": M}[case["bias"]]
        return dict(bytes=e * (M * K + K * N + M * N * (2 if case["residual"] else 1) + bias), flops=2 * M * N * K)
    if kind == "mlp":
        t, d, f = case["tokens"], case["d"], case["ffn"]
        # (the hidden activations are an output of the first call and an input of the second)
        return dict(bytes=e * (3 * t * d + 2 * t * f + 2 * d * f + d + f), flops=4 * t * d * f)
    if kind == "attention":
        b, n, d = case["bh"], case["seq"], case["d"]
        # (scores and probabilities are outputs of one call and inputs of the next: four passes over [b, n, n])
        return dict(bytes=e * b * (4 * n * d + 4 * n * n), flops=4 * b * n * n * d + 5 * b * n * n)
    if kind == "conv":
        b, ic, hw, oc, k = case["batch"], case["ic"], case["hw"], case["oc"], case["k"]
        out = (hw + 2 * case["pad"] - k) // case["stride"] + 1
        y = b * oc * out * out
        # (of a strided 1x1 convolution only the pixels that are used)
        x = b * ic * (out * out if k < case["stride"] else hw * hw)
        return dict(bytes=e * (x + oc * ic * k * k + oc + y * (2 if case["residual"] else 1)), flops=2 * y * ic * k * k)
    n = case["rows"] * case["cols"]
    if case["op"] == "softmax":
        return dict(bytes=2 * e * n, flops=5 * n)
    return dict(bytes=e * (n + case["rows"]), flops=n)


def tolerance(case):
    # Sums are fp32 whatever the storage type; what another order of them changes is the rounding of the results to it.
    # Four times what the present path differs from the same products in 64 bits: relative norm 2.8e-7 (fp32; up to 1e-6
    # where an exponential is taken), 2.2e-4 (fp16), 1.8e-3 (bf16), and for a single value 2.7e-6, 7.3e-4 and 5.9e-3.
    # Attention rounds scores before their exponential: 5.5e-4 and 8.6e-3 in fp16, eight times as much in bf16.
    if case["kind"] == "attention":
        return dict(rel=2.2e-3, max=3.5e-2) if case["dtype"] == "f16" else dict(rel=1.8e-2, max=0.28)
    return {"f32": dict(rel=4e-6, max=2e-5), "f16": dict(rel=9e-4, max=3e-3), "bf16": dict(rel=7.2e-3, max=2.4e-2)}[case["dtype"]]
