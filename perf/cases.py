"""Timed cases of the operator library: what a program that runs networks on it calls, over the sizes it calls it with.

The contractions (GEMM, batched GEMM, convolution, attention) are the library's main path; one normalisation stands for
the memory-bound operators beside them.  `listed()` has the benchmark workloads (`inputs.workload`) and the calls
around them that networks make as often: ragged sizes, a few rows against a large weight matrix (one decoding step of
several sequences), a network's first convolution with its three input channels, one query against a long key cache.
`draw()` gives further cases of the same families.
"""
from __future__ import annotations

import math

import torch

from paper_2505_02146_amd import xp

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "i8": torch.int8}
_SIZE = {"f32": 4, "bf16": 2, "i8": 1}


def listed():
    return [
        # the smallest call: a 256-cubed fp32 product, a few microseconds, where launch and latency are the time
        _gemm("f32", 256, 256, 256, "row", "row", name="gemm_f32_256"),
        # a large linear layer (activations x weights stored out x in): matrix-core bound
        _gemm("bf16", 4096, 4096, 4096, "row", "col", name="gemm_bf16_4096"),
        # A @ B with no extent a multiple of anything: sequence lengths, class counts and feature counts as data sets have them
        _gemm("bf16", 2049, 1021, 1535, "row", "row", name="gemm_bf16_odd"),
        # one decoding step of 16 sequences through a linear layer: the weights are read once, 16 rows use them
        _gemm("bf16", 16, 8192, 8192, "row", "col", name="gemm_bf16_few_rows"),
        # quantised linear layer, exact in int32
        _gemm("i8", 4096, 4096, 8192, "row", "col", name="gemm_i8_4096x4096x8192"),
        # the two products of an unfused attention block: scores (short K, large output) and weighted values (long K, narrow output)
        _bgemm(96, 512, 512, 64, "col", name="bgemm_bf16_qk"),
        _bgemm(96, 512, 64, 512, "row", name="bgemm_bf16_pv"),
        # a 3x3 stage of a residual network
        _conv(32, 56, 56, 256, 256, 3, 1, 1, name="conv_bf16_56"),
        # the first layer of such a network: three input channels, 7x7 filter, stride 2
        _conv(32, 224, 224, 3, 64, 7, 2, 3, name="conv_bf16_first_layer"),
        # attention over a prompt: 32 heads of 128
        _attention(32, 2048, 2048, 128, name="attention_bf16_2048_d128"),
        # attention of one decoding step: 8 sequences x 32 heads, one query each against 2000 cached keys
        _attention(256, 1, 2000, 128, name="attention_bf16_one_query"),
        # normalisation of a block of activations: one pass over memory
        _norm("layernorm", 16384, 4096, name="layernorm_bf16_16384x4096"),
    ]


def draw(rng):
    family = rng.choice(["f32", "bf16", "bf16", "few_rows", "i8", "scores", "values", "conv", "first_layer", "attention", "queries", "norm"])
    while True:
        case = _drawn(rng, family)
        w = work(case)
        # no more work than the largest listed case of its type
        if w["flops"] <= (4.3e9 if case.get("dtype") == "f32" else 1.4e11) and w["bytes"] <= 4e8:
            return case


# ------------------------------------------------------------------------------------------------ cases

def _gemm(dtype, M, N, K, a, b, **kw):
    return dict(kw, op="gemm", dtype=dtype, M=M, N=N, K=K, a=a, b=b)


def _bgemm(batch, M, N, K, b, **kw):
    return dict(kw, op="bgemm", batch=batch, M=M, N=N, K=K, b=b)


def _conv(n, h, w, cin, cout, r, stride, pad, **kw):
    return dict(kw, op="conv", n=n, h=h, w=w, cin=cin, cout=cout, r=r, stride=stride, pad=pad)


def _attention(batch, Lq, Lk, d, **kw):
    return dict(kw, op="attention", batch=batch, Lq=Lq, Lk=Lk, d=d)


def _norm(kind, rows, cols, **kw):
    return dict(kw, op="norm", kind=kind, rows=rows, cols=cols)


def _size(rng, lo, hi):
    """Log-uniform in lo..hi: one half as it falls, one half a multiple of 8 or, from 128 up, of 64."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        q = 64 if v >= 128 else 8
        v = max(q, v // q * q)
    return min(max(v, lo), hi)


def _drawn(rng, family):
    if family == "f32":
        return _gemm("f32", _size(rng, 16, 1024), _size(rng, 16, 1024), _size(rng, 16, 1024), "row", rng.choice(["row", "col"]))
    if family == "bf16":
        # linear layers and A @ B, and the two products of their gradients
        a, b = rng.choice([("row", "col"), ("row", "col"), ("row", "row"), ("row", "row"), ("col", "row"), ("col", "col")])
        return _gemm("bf16", _size(rng, 64, 8192), _size(rng, 64, 8192), _size(rng, 64, 8192), a, b)
    if family == "few_rows":
        return _gemm("bf16", _size(rng, 1, 64), _size(rng, 1024, 16384), _size(rng, 1024, 16384), "row", "col")
    if family == "i8":
        return _gemm("i8", _size(rng, 64, 8192), _size(rng, 64, 8192), _size(rng, 64, 8192), "row", rng.choice(["col", "col", "row"]))
    if family == "scores":
        L = _size(rng, 48, 1024)
        return _bgemm(_size(rng, 8, 192), L, L, rng.choice([32, 64, 64, 128]), "col")
    if family == "values":
        L = _size(rng, 48, 1024)
        return _bgemm(_size(rng, 8, 192), L, rng.choice([32, 64, 64, 128]), L, "row")
    if family == "conv":
        h = rng.choice([7, 14, 28, 56, 112, _size(rng, 7, 112)])
        r, s = rng.choice([(3, 1), (3, 1), (3, 2), (1, 1), (1, 2), (5, 1)])
        return _conv(_size(rng, 1, 64), h, h, _size(rng, 32, 512), _size(rng, 32, 512), r, s, r // 2)
    if family == "first_layer":
        h = _size(rng, 28, 256)
        r, s = rng.choice([(7, 2), (7, 2), (3, 1), (3, 2), (5, 1)])
        return _conv(_size(rng, 1, 64), h, h, rng.choice([3, 3, 3, 1, 4]), rng.choice([32, 64, 96]), r, s, r // 2)
    if family == "attention":
        L = _size(rng, 48, 4096)
        return _attention(_size(rng, 4, 128), L, rng.choice([L, L, _size(rng, 48, 4096)]), rng.choice([64, 128]))
    if family == "queries":
        return _attention(_size(rng, 16, 512), rng.choice([1, 1, 1, 2, 4, 8]), _size(rng, 64, 8192), rng.choice([64, 128]))
    return _norm(rng.choice(["layernorm", "rmsnorm", "softmax"]), _size(rng, 64, 16384), _size(rng, 64, 8192))


# ------------------------------------------------------------------------------------- inputs and calls

def _inputs(case, seed):
    """The operands, on the GPU: contractions of N(0, 1) values scaled as trained layers are, so that outputs are of order one."""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, scale=1.0):
        return (torch.randn(*shape, device="cuda", generator=g) * scale).bfloat16()

    op = case["op"]
    if op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        sa, sb = ((M, K) if case["a"] == "row" else (K, M)), ((K, N) if case["b"] == "row" else (N, K))
        if case["dtype"] == "i8":
            return [torch.randint(-128, 128, s, device="cuda", dtype=torch.int8, generator=g) for s in (sa, sb)]
        if case["dtype"] == "f32":
            return [torch.rand(s, device="cuda", generator=g) * 2 - 1 for s in (sa, sb)]
        return [normal(*sa), normal(*sb, scale=K ** -0.5)]
    if op == "bgemm":
        b, M, N, K = case["batch"], case["M"], case["N"], case["K"]
        return [normal(b, M, K, scale=0.125), normal(*((b, K, N) if case["b"] == "row" else (b, N, K)), scale=0.125)]
    if op == "conv":
        r, cin = case["r"], case["cin"]
        return [normal(case["n"], case["h"], case["w"], cin), normal(case["cout"], r, r, cin, scale=(r * r * cin) ** -0.5)]
    if op == "attention":
        b, d = case["batch"], case["d"]
        return [normal(b, case["Lq"], d), normal(b, case["Lk"], d), normal(b, case["Lk"], d)]
    cols = case["cols"]
    return [normal(case["rows"], cols), normal(cols), normal(cols)]


def _out_shape(case):
    op = case["op"]
    if op == "gemm":
        return case["M"], case["N"]
    if op == "bgemm":
        return case["batch"], case["M"], case["N"]
    if op == "conv":
        p, q = ((case[e] + 2 * case["pad"] - case["r"]) // case["stride"] + 1 for e in ("h", "w"))
        return case["n"], p, q, case["cout"]
    if op == "attention":
        return case["batch"], case["Lq"], case["d"]
    return case["rows"], case["cols"]


def _out_type(case):
    if case["op"] == "norm":
        return torch.bfloat16
    return torch.int32 if case.get("dtype") == "i8" else torch.float32


def prepare(case, seed):
    return dict(case=case, x=_inputs(case, seed), out=torch.empty(_out_shape(case), device="cuda", dtype=_out_type(case)))


def run(state):
    case, x, out = state["case"], state["x"], state["out"]
    op = case["op"]
    if op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        xp.xp_gemm(M, N, K, 1.0, x[0], case["a"], K if case["a"] == "row" else M, x[1], case["b"], N if case["b"] == "row" else K,
                   0.0, out, "row", N)
    elif op == "bgemm":
        M, N, K = case["M"], case["N"], case["K"]
        xp.xp_gemm_batched(case["batch"], M, N, K, 1.0, x[0], "row", K, M * K, x[1], case["b"], N if case["b"] == "row" else K,
                           K * N, 0.0, out, "row", N, M * N)
    elif op == "conv":
        xp.xp_conv2d_nhwc(case["n"], case["h"], case["w"], case["cin"], case["cout"], case["r"], case["r"], case["stride"],
                          case["stride"], case["pad"], case["pad"], x[0], x[1], "krsc", out)
    elif op == "attention":
        Lq, Lk, d = case["Lq"], case["Lk"], case["d"]
        xp.xp_attention(case["batch"], Lq, Lk, d, d, d ** -0.5, x[0], d, Lq * d, x[1], d, Lk * d, x[2], d, Lk * d, out, d, Lq * d)
    elif case["kind"] == "layernorm":
        xp.xp_layernorm(case["rows"], case["cols"], x[0], case["cols"], x[1], x[2], 1e-5, out, case["cols"])
    elif case["kind"] == "rmsnorm":
        xp.xp_rmsnorm(case["rows"], case["cols"], x[0], case["cols"], x[1], 1e-6, out, case["cols"])
    else:
        xp.xp_softmax(case["rows"], case["cols"], x[0], case["cols"], out, case["cols"])
    return out


# ------------------------------------------------------------------------------- work, tolerance, exact

def work(case):
    op = case["op"]
    outputs = math.prod(_out_shape(case))
    if op in ("gemm", "bgemm"):
        M, N, K, b = case["M"], case["N"], case["K"], case.get("batch", 1)
        return {"bytes": b * (M * K + K * N) * _SIZE[case.get("dtype", "bf16")] + 4 * outputs, "flops": 2 * b * M * N * K}
    if op == "conv":
        taps = case["r"] * case["r"] * case["cin"]
        return {"bytes": 2 * (case["n"] * case["h"] * case["w"] * case["cin"] + taps * case["cout"]) + 4 * outputs, "flops": 2 * outputs * taps}
    if op == "attention":
        b, Lq, Lk, d = case["batch"], case["Lq"], case["Lk"], case["d"]
        return {"bytes": 2 * b * d * (Lq + 2 * Lk) + 4 * outputs, "flops": 4 * b * Lq * Lk * d}
    vectors = {"layernorm": 2, "rmsnorm": 1, "softmax": 0}[case["kind"]]
    return {"bytes": 2 * outputs + 2 * vectors * case["cols"] + 2 * outputs, "flops": 8 * outputs}


def tolerance(case):
    if case.get("dtype") == "i8":
        return "exact"
    if case["op"] == "norm":
        return {"rel": 7e-3}          # bf16 results: 1.7e-3 from the rounding alone
    if case["op"] == "attention":
        return {"rel": 7e-3}          # probabilities may be rounded to bf16 before they meet V: 1.6e-3
    return {"rel": 3e-6}              # exact products, sums in fp32


def exact(case, seed):
    x = _inputs(case, seed)
    op = case["op"]
    if op == "norm":
        v = x[0].double()
        if case["kind"] == "softmax":
            return torch.softmax(v, -1)
        if case["kind"] == "rmsnorm":
            return v / (v.square().mean(-1, keepdim=True) + 1e-6).sqrt() * x[1].double()
        v = v - v.mean(-1, keepdim=True)
        return v / (v.square().mean(-1, keepdim=True) + 1e-5).sqrt() * x[1].double() + x[2].double()
    x = [t.double() for t in x]
    if op == "gemm":
        r = (x[0] if case["a"] == "row" else x[0].t().contiguous()) @ (x[1] if case["b"] == "row" else x[1].t().contiguous())
        return r.to(torch.int32) if case["dtype"] == "i8" else r
    if op == "bgemm":
        return torch.bmm(x[0], x[1] if case["b"] == "row" else x[1].transpose(1, 2).contiguous())
    if op == "conv":
        n, p, q, cout = _out_shape(case)
        s, pad = case["stride"], case["pad"]
        image = torch.nn.functional.pad(x[0], (0, 0, pad, pad, pad, pad))
        out = torch.zeros(n * p * q, cout, device="cuda", dtype=torch.float64)
        for i in range(case["r"]):
            for j in range(case["r"]):
                tap = image[:, i:i + s * (p - 1) + 1:s, j:j + s * (q - 1) + 1:s, :].reshape(n * p * q, case["cin"])
                out += tap @ x[1][:, i, j, :].t().contiguous()
        return out.reshape(n, p, q, cout)
    out = []
    for first in range(0, case["batch"], 8):
        qs, ks, vs = (t[first:first + 8] for t in x)
        scores = torch.bmm(qs, ks.transpose(1, 2).contiguous()) * case["d"] ** -0.5
        out.append(torch.bmm(torch.softmax(scores, -1), vs))
    return torch.cat(out)
