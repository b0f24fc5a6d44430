"""What the choice among the kernel variants costs: random calls, every variant that takes a call timed beside the one that the
library chooses.  The figures beside the fitted times (`csrc/xp_api.hip`) and the estimate for rows of any alignment
(`csrc/xp_mfma_ua.hpp`) are of this kind.

    python -m paper_2505_02146_amd.time_variants --calls 1000 [--seed 1] [--families gemm_bf16 ...] [--align aligned|any]
        [--out calls.jsonl]
    python -m paper_2505_02146_amd.time_variants --compare before.jsonl after.jsonl

A line of the output is a call, the chosen variant and each variant's microseconds.  `--compare` takes the same calls (seed and
number) from two builds and sets the second's choice against the first's, both by the second's timings.
"""
from __future__ import annotations

import argparse
import json
import math
import random

FAMILIES = ("gemm_bf16", "gemm_i8", "batched_bf16", "batched_i8", "conv")
MAX_FLOPS, MAX_OPERAND, MAX_OUT = 1.4e11, 1 << 27, 1 << 26           # operations; elements of one operand and of the output


def _size(rng, lo, hi, step):
    """Log-uniform in lo..hi, a multiple of `step`, one half of those from 128 up a multiple of 64."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    q = 64 if v >= 128 and rng.random() < 0.5 else step
    return max(q, int(v) // q * q)


def draw(rng, family, align):
    """One call of `family`; align "aligned": rows of whole 16 bytes (convolution: channels of whole 64 bytes), "any": any extent."""
    step = 1 if align == "any" else (16 if family.endswith("i8") else 8)
    while True:
        if family == "conv":
            r, s = rng.choice([(3, 1), (3, 1), (3, 2), (1, 1), (1, 2), (5, 1)])
            h = rng.choice([7, 14, 28, 56, 112])
            cin = _size(rng, 32, 512, 1 if align == "any" else 32)
            c = dict(family=family, n=_size(rng, 1, 64, 1), h=h, cin=cin, cout=_size(rng, 32, 512, 1), r=r, stride=s, pad=r // 2)
            p = (h + 2 * c["pad"] - r) // s + 1
            out, a, b = c["n"] * p * p * c["cout"], c["n"] * h * h * cin, c["cout"] * r * r * cin
            flops = 2.0 * out * r * r * cin
        else:
            if family.startswith("batched"):
                L, d = _size(rng, 48, 1024, step), rng.choice([32, 64, 64, 128])
                M, N, K = rng.choice([(L, L, d), (L, d, L)])
                batch = _size(rng, 8, 192, 1)
            else:
                M, N, K, batch = _size(rng, 64, 8192, step), _size(rng, 64, 8192, step), _size(rng, 64, 8192, step), 0
            c = dict(family=family, batch=batch, M=M, N=N, K=K, a=rng.choice(["row", "row", "col"]), b=rng.choice(["row", "col"]))
            n = max(batch, 1)
            out, a, b = n * M * N, n * M * K, n * N * K
            flops = 2.0 * out * K
        if flops <= MAX_FLOPS and max(a, b) <= MAX_OPERAND and out <= MAX_OUT:
            return c


class Runner:
    """Operands and output of the largest call; a call takes their beginnings."""

    def __init__(self, torch, xp):
        self.torch, self.xp = torch, xp
        g = torch.Generator(device="cuda").manual_seed(0)
        self.bf16 = [torch.randn(MAX_OPERAND, device="cuda", generator=g).bfloat16() for _ in range(2)]
        self.i8 = [torch.randint(-128, 128, (MAX_OPERAND,), device="cuda", dtype=torch.int8, generator=g) for _ in range(2)]
        self.out = torch.zeros(MAX_OUT, device="cuda")

    def call(self, c):
        """(operator, type, function that runs the call once)"""
        xp = self.xp
        if c["family"] == "conv":
            a, b = self.bf16
            return xp.XP_OP_CONV2D, "bf16", lambda: xp.xp_conv2d_nhwc(
                c["n"], c["h"], c["h"], c["cin"], c["cout"], c["r"], c["r"], c["stride"], c["stride"], c["pad"], c["pad"], a, b, "krsc", self.out)
        kind = "i8" if c["family"].endswith("i8") else "bf16"
        a, b = self.i8 if kind == "i8" else self.bf16
        out = self.out.view(self.torch.int32) if kind == "i8" else self.out
        M, N, K = c["M"], c["N"], c["K"]
        lda, ldb = K if c["a"] == "row" else M, N if c["b"] == "row" else K
        if c["batch"]:
            return xp.XP_OP_GEMM_BATCHED, kind, lambda: xp.xp_gemm_batched(
                c["batch"], M, N, K, 1.0, a, c["a"], lda, M * K, b, c["b"], ldb, N * K, 0.0, out, "row", N, M * N)
        return xp.XP_OP_GEMM, kind, lambda: xp.xp_gemm(M, N, K, 1.0, a, c["a"], lda, b, c["b"], ldb, 0.0, out, "row", N)

    def burst(self, fn, n):
        e0, e1 = (self.torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        for _ in range(n):
            fn()
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / n * 1e3

    def time(self, c, bursts=3):
        """The chosen variant's name, and microseconds by name: the shortest of three bursts, the variants in turns."""
        xp = self.xp
        op, kind, fn = self.call(c)
        xp.xp_force_config(op, kind, -1)
        fn()
        chosen = xp.xp_last_config(op, kind)
        us = {}
        try:
            for v in range(xp.xp_num_configs(op, kind)):
                if v == 0 and chosen != 0:                        # the general kernel: up to a hundred times the others' time
                    continue
                xp.xp_force_config(op, kind, v)
                try:
                    fn()
                except xp.XpError:
                    continue
                us[v] = math.inf
            for _ in range(bursts):
                for v in us:
                    xp.xp_force_config(op, kind, v)
                    once = self.burst(fn, 2)
                    us[v] = min(us[v], self.burst(fn, max(5, min(40, int(400 / once)))))
        finally:
            xp.xp_force_config(op, kind, -1)
        return xp.xp_describe_config(op, kind, chosen), {xp.xp_describe_config(op, kind, v): round(t, 3) for v, t in us.items()}


def summary(calls):
    """Lines on the chosen variants' times over the best ones', by family."""
    lines = []
    for f in (*FAMILIES, "all"):
        over = sorted(c["us"][c["chosen"]] / min(c["us"].values()) for c in calls if f in ("all", c["family"]))
        if over:
            lines.append(f"{f}: {len(over)} calls, the chosen variant over the best: geometric mean {math.exp(sum(map(math.log, over)) / len(over)):.3f}, "
                         f"{sum(x > 1.05 for x in over)} more than 5 % slower, {sum(x > 1.2 for x in over)} more than 20 %, worst {over[-1]:.2f}")
    return lines


def compare(before, after):
    """Lines on the choices that differ between two builds' runs over the same calls."""
    key = lambda c: json.dumps({k: v for k, v in c.items() if k not in ("chosen", "us")}, sort_keys=True)
    old = {key(c): c["chosen"] for c in before}
    ratio = sorted((c["us"][c["chosen"]] / c["us"][old[key(c)]], key(c)) for c in after
                   if old.get(key(c), c["chosen"]) != c["chosen"] and old[key(c)] in c["us"])
    return [f"{sum(key(c) in old for c in after)} calls in both, {len(ratio)} choices differ: {sum(r < 1 / 1.05 for r, _ in ratio)} more than 5 % faster, "
            f"{sum(r > 1.05 for r, _ in ratio)} more than 5 % slower"] + [f"  x{r:.2f} {k}" for r, k in ratio[-10:] if r > 1.05]


def main(argv=None) -> int:
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--calls", type=int, default=200)
    ap.add_argument("--seed", type=int, default=1)
    ap.add_argument("--families", nargs="*", choices=FAMILIES, default=list(FAMILIES))
    ap.add_argument("--align", choices=("aligned", "any"), default="aligned")
    ap.add_argument("--out")
    ap.add_argument("--compare", nargs=2, metavar=("BEFORE", "AFTER"))
    args = ap.parse_args(argv)
    if args.compare:
        runs = [[json.loads(line) for line in open(name)] for name in args.compare]
        print("\n".join(compare(*runs)))
        return 0
    import torch
    from . import xp
    rng = random.Random(args.seed)
    drawn = [draw(rng, rng.choice(args.families), args.align) for _ in range(args.calls)]
    runner, calls = Runner(torch, xp), []
    out = open(args.out, "w") if args.out else None
    for i, c in enumerate(drawn):
        if i % 100 == 0:
            print(f"call {i}: {c}", flush=True)
        chosen, us = runner.time(c)
        calls.append(dict(c, chosen=chosen, us=us))
        if out:
            out.write(json.dumps(calls[-1]) + "\n")
            out.flush()
    print("\n".join(summary(calls)))
    return 0


if __name__ == "__main__":
    raise SystemExit(main())
