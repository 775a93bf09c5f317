"""What a user of this package has it do, as cases that can be timed and compared: whole paths through the public entry
points of paper_2408_02897_amd.qmm and .experiments, over the sizes the package's own configurations name (BERT-base and
BERT-large linear layers, their backward products, attention, the 512 x 512 example) and the odd ones in between.

  linear     one quantized product as the method defines it: step size and codes of both operands, product, error
             metric against a high-precision product that is in hand
  layer      the four forward products of a transformer layer through the several-tensors calls and kept buffers, as the
             benchmark's step has them
  backward   the two backward products of a linear layer (both operands' transposes are made by the quantize pass)
  attention  the two batched products of attention with one step size per head
  gemm       a product of code matrices that are in hand
  reference  the high-precision product
  example    the backward-error example: one step size per vector, product, reference, |L| |R|, metric with denominators
  stats      what is looked at before a format is chosen: moments, and the error of quantizing the tensor itself
  choose     the error of every candidate format on one product
"""
import math

import numpy as np
import torch

from paper_2408_02897_amd import experiments, qmm

DEV = "cuda"
FMT = {"int8": qmm.INT8, "e4m3": qmm.E4M3, "e5m2": qmm.E5M2}
QMAX = {"int8": 127.0, "e4m3": 448.0, "e5m2": 57344.0}
MANTISSA = {"e4m3": (3, -6), "e5m2": (2, -14)}          # mantissa bits, exponent of the smallest normal value
DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # the smallest whole call: a single linear layer, 256 tokens; latency and launches
        dict(name="linear small", kind="linear", m=256, n=768, k=768, fmt="e4m3", channel=False, src="bf16", out="f32", mode="rtne", pad=0),
        # a float32 model (as the reference BERT is kept) with ragged token and feature counts, step sizes per channel
        dict(name="linear ragged f32", kind="linear", m=1031, n=1000, k=784, fmt="e4m3", channel=True, src="f32", out="f32", mode="rtne", pad=0),
        # BERT-base FFN1 at batch 32 x 128, INT8 with step sizes per channel
        dict(name="linear base int8", kind="linear", m=4096, n=3072, k=768, fmt="int8", channel=True, src="bf16", out="bf16", mode="rtne", pad=0),
        # BERT-large forward, one layer, batch 32 x 512
        dict(name="layer large", kind="layer", m=16384, hidden=1024, ffn=4096, fmt="e4m3"),
        # BERT-base FFN2 backward, step sizes per channel, gradients rounded stochastically
        dict(name="backward base sr", kind="backward", m=4096, n=768, k=3072, fmt="e4m3", grad="e5m2", channel=True, src="bf16", mode="sr"),
        # BERT-large QKV backward, step sizes per tensor
        dict(name="backward large", kind="backward", m=16384, n=3072, k=1024, fmt="e4m3", grad="e5m2", channel=False, src="bf16", mode="rtne"),
        # BERT-large attention, batch 32, one step size per head
        dict(name="attention large", kind="attention", examples=32, heads=16, seq=512, dim=64, fmt="e4m3"),
        # BERT-large FFN2 on codes in hand
        dict(name="gemm large int8", kind="gemm", m=16384, n=1024, k=4096, fmt="int8", fmt_b="int8", channel=True, out="bf16"),
        # the high-precision product of BERT-large FFN1
        dict(name="reference large", kind="reference", m=16384, n=4096, k=1024),
        # the 512 x 512 Student-t example, one step size per vector
        dict(name="example 512", kind="example", n=512, dof=3, fmt="e4m3"),
        # BERT-large FFN2's activations: moments, and the relative error of the quantized values
        dict(name="stats large", kind="stats", m=16384, k=4096, fmt="e4m3", channel=False, src="bf16"),
        # format x granularity on BERT-base's attention output projection
        dict(name="choose base", kind="choose", m=4096, n=768, k=768),
    ]


def _log(rng, lo, hi, of=1):
    """A multiple of `of` in [lo, hi], spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / of)) * of))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "backward", "backward", "attention", "gemm", "gemm", "reference",
                       "example", "stats", "layer", "choose"])
    pick = rng.choice
    if kind == "linear":
        return dict(kind=kind, m=_log(rng, 64, 16384, pick([1, 1, 32])), n=_log(rng, 128, 4096, pick([1, 8, 64])), k=_log(rng, 256, 4096, 16),
                    fmt=pick(["int8", "e4m3", "e4m3", "e5m2"]), channel=pick([True, False]), src=pick(["bf16", "bf16", "f32"]),
                    out=pick(["bf16", "f32"]), mode=pick(["rtne", "rtne", "rtne", "sr"]), pad=pick([0, 0, 0, 64]))
    if kind == "backward":
        fmt = pick(["e4m3", "e4m3", "int8"])
        return dict(kind=kind, m=_log(rng, 256, 16384, 16), n=_log(rng, 128, 4096, 16), k=_log(rng, 128, 4096, pick([1, 8, 64])), fmt=fmt,
                    grad="int8" if fmt == "int8" else "e5m2", channel=pick([True, False]), src=pick(["bf16", "bf16", "f32"]),
                    mode=pick(["rtne", "rtne", "sr"]))
    if kind == "attention":
        return dict(kind=kind, examples=_log(rng, 1, 32), heads=pick([12, 16]), seq=_log(rng, 64, 512, 16), dim=64, fmt=pick(["e4m3", "int8"]))
    if kind == "gemm":
        fmt = pick(["int8", "e4m3", "e5m2"])
        return dict(kind=kind, m=_log(rng, 128, 16384, pick([1, 64, 256])), n=_log(rng, 128, 4096, pick([1, 64, 256])), k=_log(rng, 256, 8192, 16), fmt=fmt,
                    fmt_b="int8" if fmt == "int8" else pick(["e4m3", "e5m2"]), channel=pick([True, False]), out=pick(["bf16", "f32"]))
    if kind == "reference":
        return dict(kind=kind, m=_log(rng, 128, 16384, pick([1, 64])), n=_log(rng, 128, 4096, pick([1, 64])), k=_log(rng, 256, 4096, 16))
    if kind == "example":
        return dict(kind=kind, n=_log(rng, 128, 1024, 16), dof=pick([1, 2, 3, 4, 6, 10, 30]), fmt=pick(["int8", "e4m3", "e5m2"]))
    if kind == "stats":
        return dict(kind=kind, m=_log(rng, 256, 16384), k=_log(rng, 256, 4096, pick([1, 8, 64])), fmt=pick(["int8", "e4m3", "e5m2"]),
                    channel=pick([True, False]), src=pick(["bf16", "bf16", "f32"]))
    if kind == "layer":
        hidden = pick([256, 512, 768, 1024])
        return dict(kind=kind, m=_log(rng, 128, 16384, pick([1, 128])), hidden=hidden, ffn=4 * hidden, fmt=pick(["e4m3", "int8", "e5m2"]))
    return dict(kind="choose", m=_log(rng, 256, 8192, pick([1, 64])), n=_log(rng, 256, 3072, pick([1, 64])), k=_log(rng, 256, 3072, 16))


# ---------------------------------------------------------------------------------------------------- inputs
class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, shape, std=1.0):
        return torch.randn(shape, generator=self.g, device=DEV) * std

    def student_t(self, shape, dof):                      # activations: heavy tails
        z, chi2 = self.normal(shape), torch.zeros(shape, device=DEV)
        for _ in range(dof):
            chi2 += self.normal(shape).square_()
        return z / (chi2 / dof).sqrt()

    def gradient(self, shape):                            # upstream gradients: log-normal magnitudes, fair signs
        sign = (torch.rand(shape, generator=self.g, device=DEV) < 0.5).float() * 2 - 1
        return sign * torch.exp(self.normal(shape, 2.0) - 8.0)


def _layer_ops(case):
    m, h, f = case["m"], case["hidden"], case["ffn"]
    return [(m, 3 * h, h), (m, h, h), (m, f, h), (m, h, f)]


def _reference(x, w):
    return (x.float() @ w.float().t()).unsqueeze(0)


def prepare(case, seed):
    d, s, kind = _Draws(seed), {"case": case, "seed": seed}, case["kind"]
    if kind == "linear":
        t = DTYPE[case["src"]]
        s["x"] = d.student_t((case["m"], case["k"] + case["pad"]), 4).to(t)[:, :case["k"]]
        s["w"] = d.normal((case["n"], case["k"]), 0.02).to(t)
        s["ref"] = _reference(s["x"], s["w"])
    elif kind == "layer":
        s["ops"] = []
        for m, n, k in _layer_ops(case):
            x, w = d.student_t((m, k), 4).bfloat16(), d.normal((n, k), 0.02).bfloat16()
            o = dict(x=x, w=w, ref=_reference(x, w), desc=qmm.MultiDesc([x, w]))
            o["delta"] = [torch.empty(1, device=DEV) for _ in range(2)]
            o["codes"] = [torch.empty((1,) + tuple(t.shape), dtype=torch.uint8, device=DEV) for t in (x, w)]
            o["y"] = torch.empty((1, m, n), dtype=torch.bfloat16, device=DEV)
            o["operands"] = [qmm.operand(c, FMT[case["fmt"]], dl) for c, dl in zip(o["codes"], o["delta"])]
            s["ops"].append(o)
    elif kind == "backward":
        t = DTYPE[case["src"]]
        s["x"] = d.student_t((case["m"], case["k"]), 4).to(t)
        s["w"] = d.normal((case["n"], case["k"]), 0.02).to(t)
        s["dy"] = d.gradient((case["m"], case["n"])).to(t)
    elif kind == "attention":
        shape = (case["examples"], case["heads"], case["seq"], case["dim"])
        q, k, v = (d.normal(shape) for _ in range(3))
        channels = case["heads"] * case["dim"]            # one channel in a hundred is an outlier, as the heads of trained models have
        out = torch.randperm(channels, generator=d.g, device=DEV)[:max(1, channels // 100)]
        gain = torch.ones(channels, device=DEV)
        gain[out] = 20.0
        gain = gain.view(1, case["heads"], 1, case["dim"])
        s["q"], s["k"], s["v"] = ((t * gain).bfloat16().view(-1, case["seq"], case["dim"]) for t in (q, k, v))
        scores = s["q"].float() @ s["k"].float().transpose(1, 2).contiguous()
        s["p"] = torch.softmax(scores / math.sqrt(case["dim"]), dim=-1).bfloat16()
    elif kind == "gemm":
        x, w = d.student_t((case["m"], case["k"]), 4).bfloat16(), d.normal((case["n"], case["k"]), 0.02).bfloat16()
        s["a"], s["da"] = qmm.quantized_operand(x, 1, FMT[case["fmt"]], case["channel"])
        s["b"], s["db"] = qmm.quantized_operand(w, 1, FMT[case["fmt_b"]], case["channel"])
    elif kind == "example":
        s["l"], s["r"] = (d.student_t((case["n"], case["n"]), case["dof"]).bfloat16() for _ in range(2))
        s["l_abs"], s["r_abs"] = s["l"].abs(), s["r"].abs()
    elif kind == "stats":
        s["x"] = d.student_t((case["m"], case["k"]), 4).to(DTYPE[case["src"]])
        s["x32"] = s["x"].float()
    else:                                                 # reference, choose
        s["x"] = d.student_t((case["m"], case["k"]), 4).bfloat16()
        s["w"] = d.normal((case["n"], case["k"]), 0.02).bfloat16()
    return s


# ---------------------------------------------------------------------------------------------------- one pass
def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "linear":
        fmt, mode = FMT[case["fmt"]], qmm.STOCHASTIC if case["mode"] == "sr" else qmm.RTNE
        a, dx = qmm.quantized_operand(s["x"], 1, fmt, case["channel"], mode=mode, seed=s["seed"])
        b, dw = qmm.quantized_operand(s["w"], 1, fmt, case["channel"])
        y = qmm.gemm(a, b, DTYPE[case["out"]])
        return dict(y=y, dx=dx, dw=dw, metric=qmm.metric(y, s["ref"]))
    if kind == "layer":
        fmt, out = FMT[case["fmt"]], []
        for o in s["ops"]:
            qmm.scale_multi(o["desc"], fmt, outs=o["delta"])
            qmm.quantize_multi(o["desc"], fmt, o["delta"], outs=o["codes"])
            y = qmm.gemm((o["codes"][0], o["operands"][0]), (o["codes"][1], o["operands"][1]), out=o["y"])
            out.append(dict(y=y, metric=qmm.metric(y, o["ref"]), delta=list(o["delta"])))
        return out
    if kind == "backward":
        fmt, grad, ch = FMT[case["fmt"]], FMT[case["grad"]], case["channel"]
        mode = qmm.STOCHASTIC if case["mode"] == "sr" else qmm.RTNE
        dy_n, _ = qmm.quantized_operand(s["dy"], 1, grad, ch, mode=mode, seed=s["seed"])
        w_n, _ = qmm.quantized_operand(s["w"], 0, fmt, ch)
        dx = qmm.gemm(dy_n, w_n, torch.bfloat16)
        dy_m, _ = qmm.quantized_operand(s["dy"], 0, grad, ch, mode=mode, seed=s["seed"] + 1)
        x_m, _ = qmm.quantized_operand(s["x"], 0, fmt, ch)
        return dict(dx=dx, dw=qmm.gemm(dy_m, x_m, torch.float32))
    if kind == "attention":
        fmt, heads = FMT[case["fmt"]], case["heads"]
        q, _ = qmm.quantized_operand(s["q"], 1, fmt, batch_groups=heads)
        k, _ = qmm.quantized_operand(s["k"], 1, fmt, batch_groups=heads)
        scores = qmm.gemm(q, k, torch.bfloat16)
        p, _ = qmm.quantized_operand(s["p"], 1, fmt, batch_groups=heads)
        v, _ = qmm.quantized_operand(s["v"], 0, fmt, batch_groups=heads)
        return dict(scores=scores, out=qmm.gemm(p, v, torch.bfloat16))
    if kind == "gemm":
        return dict(y=qmm.gemm(s["a"], s["b"], DTYPE[case["out"]]))
    if kind == "reference":
        return dict(y=qmm.reference_gemm(s["x"].unsqueeze(0), s["w"].unsqueeze(0)))
    if kind == "example":
        fmt = FMT[case["fmt"]]
        a, _ = qmm.quantized_operand(s["l"], 1, fmt, per_channel=True)
        b, _ = qmm.quantized_operand(s["r"], 1, fmt, per_channel=True)
        y = qmm.gemm(a, b, torch.float32)
        ref = qmm.reference_gemm(s["l"].unsqueeze(0), s["r"].unsqueeze(0))
        denom = qmm.reference_gemm(s["l_abs"].unsqueeze(0), s["r_abs"].unsqueeze(0))
        m = qmm.metric(y, ref, denom)
        # without the sum and maximum of |e| / |ref|, which hang on the last bits of the reference's smallest element
        return dict(y=y, ref=ref, denom=denom, sums=m[0:6], backward=m[8:16])
    if kind == "stats":
        fmt, ch = FMT[case["fmt"]], case["channel"]
        moments = qmm.moments(s["x"])
        delta = qmm.scale(s["x"], 1, fmt, ch)
        codes = qmm.quantize(s["x"], 1, fmt, delta, ch)
        values = qmm.dequantize(codes[0], fmt, delta, ch)
        return dict(moments=moments, delta=delta, codes=codes, values=values, metric=qmm.metric(values, s["x32"]))
    rows = experiments.format_sweep(s["x"], s["w"])
    # (again without the |e| / |ref| of the reference's smallest elements)
    return [np.array([r["nsr"]] + [r["fields"][f] for f in ("S_ee", "S_rr", "S_ae", "S_ar", "M_e", "M_r", "n")]) for r in rows]


# ---------------------------------------------------------------------------------------------------- sizes
def work(case):
    kind, out = case["kind"], {"bf16": 2, "f32": 4}.get(case.get("out"), 0)
    src = {"bf16": 2, "f32": 4}.get(case.get("src"), 2)
    m, n, k = case.get("m"), case.get("n"), case.get("k")
    if kind == "linear":
        return dict(bytes=src * (m + n) * k + (out + 4) * m * n, flops=2 * m * n * k)
    if kind == "layer":
        ops = _layer_ops(case)
        return dict(bytes=sum(2 * (a + b) * c + 6 * a * b for a, b, c in ops), flops=sum(2 * a * b * c for a, b, c in ops))
    if kind == "backward":
        return dict(bytes=src * (m * k + n * k + m * n) + 2 * m * k + 4 * n * k, flops=4 * m * n * k)
    if kind == "attention":
        b, s, d = case["examples"] * case["heads"], case["seq"], case["dim"]
        return dict(bytes=2 * b * (3 * s * d + s * s) + 2 * b * (s * s + s * d), flops=4 * b * s * s * d)
    if kind == "gemm":
        return dict(bytes=(m + n) * k + out * m * n, flops=2 * m * n * k)
    if kind == "reference":
        return dict(bytes=2 * (m + n) * k + 4 * m * n, flops=2 * m * n * k)
    if kind == "example":
        return dict(bytes=8 * n * n + 12 * n * n, flops=6 * n ** 3)
    if kind == "stats":
        return dict(bytes=(src + 4 + 1 + 4) * m * k, flops=0)
    return dict(bytes=2 * (m + n) * k, flops=14 * m * n * k)


def tolerance(case):
    """Measured against exact(), times about four: FP8 products 2e-5 off on activations and weights and 7e-5 on log-normal
    gradients (the matrix unit's own sums), the reference product 2e-7, binary64 sums over equal inputs 1e-9; bfloat16
    results may be the neighbouring value now and then."""
    kind = case["kind"]
    if kind in ("linear", "layer", "gemm", "backward", "attention"):
        return dict(rel=3e-4, max=4e-3) if case.get("out") == "f32" else dict(rel=1e-3, max=1.6e-2)
    if kind == "stats":
        return dict(rel=1e-9, max=1e-9)                   # whole codes are the same
    if kind == "reference":
        return dict(rel=2e-6, max=5e-5)
    return dict(rel=1e-4, max=2e-3)


# ---------------------------------------------------------------------------------------------------- in 64 bits
def _philox_u24(count, seed):
    """The 24 random bits of elements 0 .. count - 1: Philox4x32-10, counter = element / 4, word = element % 4."""
    mask = 0xFFFFFFFF
    blk = torch.arange((count + 3) // 4, dtype=torch.int64, device=DEV)
    c0, c1 = blk & mask, blk >> 32
    c2, c3, k0, k1 = torch.zeros_like(blk), torch.zeros_like(blk), seed & mask, (seed >> 32) & mask
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask
    return torch.stack((c0, c1, c2, c3), dim=1).reshape(-1)[:count] >> 8


def _quantized(x, axis, fmt, channel=False, groups=1, sr_seed=None):
    """(values of the codes, step sizes) with the contracting axis last: the step size is a binary32 quotient, a code
    the rounding of a binary32 product, as the method's call defines them; the values are binary64."""
    x = (x if x.dim() == 3 else x.unsqueeze(0)).float()
    if axis == 0:
        x = x.transpose(1, 2).contiguous()
    b, n, k = x.shape
    by = x.abs().view(b // groups, groups, n, k)
    a = by.amax(dim=(0, 3), keepdim=True) if channel else by.amax(dim=(0, 2, 3), keepdim=True)
    # (a tensor as the divisor: by a number, the GPU would multiply with its rounded reciprocal)
    delta = torch.where(a == 0, torch.ones_like(a), (a / torch.full_like(a, QMAX[fmt])).clamp(min=2.0 ** -126))
    t = (x.view(b // groups, groups, n, k) * (1.0 / delta)).view(b, n, k)
    if sr_seed is not None:
        mag = t.abs().double().clamp(max=QMAX[fmt])
        if fmt == "int8":
            step = torch.ones_like(mag)
        else:
            bits, low = MANTISSA[fmt]
            step = torch.exp2((torch.frexp(mag).exponent - 1).clamp(min=low).double() - bits)
        lo = torch.floor(mag / step)
        up = _philox_u24(x.numel(), sr_seed).view(b, n, k).double() < (mag / step - lo) * 2.0 ** 24
        v = torch.sign(t).double() * torch.minimum((lo + up) * step, torch.full_like(mag, QMAX[fmt]))
    elif fmt == "int8":
        v = torch.round(t).clamp(-127, 127).double()
    else:
        v = t.clamp(-QMAX[fmt], QMAX[fmt]).to(torch.float8_e4m3fn if fmt == "e4m3" else torch.float8_e5m2).double()
    return v, delta.double().view(1, groups, -1, 1).expand(b // groups, groups, n if channel else 1, 1).reshape(b, -1, 1), delta.view(-1).double()


def _product(a, b):
    return (a[0] @ b[0].transpose(1, 2).contiguous()) * a[1] * b[1].transpose(1, 2)


def _metric(y, r, d=None):
    y, r = y.double().reshape(-1), r.double().reshape(-1)
    e, a = (y - r).abs(), r.abs()
    q = torch.where(a > 0, e / a, torch.zeros_like(e))
    z = torch.zeros((), dtype=torch.float64, device=DEV)
    m = [e.square().sum(), a.square().sum(), e.sum(), a.sum(), e.max(), a.max(), q.sum(), q.max(), (a > 0).sum().double(), z, z, z,
         z + y.numel(), z, z, z]
    if d is not None:
        d = d.double().reshape(-1)
        q = torch.where(d > 0, e / d, torch.zeros_like(e))
        m[9:12] = [q.sum(), q.max(), (d > 0).sum().double()]
    return torch.stack(m)


def exact(case, seed):
    s, kind, fmt = prepare(case, seed), case["kind"], case.get("fmt")
    sr = seed if case.get("mode") == "sr" else None
    if kind == "linear":
        a, b = _quantized(s["x"], 1, fmt, case["channel"], sr_seed=sr), _quantized(s["w"], 1, fmt, case["channel"])
        y = _product(a, b)
        return dict(y=y, dx=a[2], dw=b[2], metric=_metric(y.to(DTYPE[case["out"]]), s["ref"]))
    if kind == "layer":
        out = []
        for o in s["ops"]:
            a, b = _quantized(o["x"], 1, fmt), _quantized(o["w"], 1, fmt)
            y = _product(a, b)
            out.append(dict(y=y, metric=_metric(y.bfloat16(), o["ref"]), delta=[a[2], b[2]]))
        return out
    if kind == "backward":
        ch = case["channel"]
        dx = _product(_quantized(s["dy"], 1, case["grad"], ch, sr_seed=sr), _quantized(s["w"], 0, fmt, ch))
        dw = _product(_quantized(s["dy"], 0, case["grad"], ch, sr_seed=None if sr is None else sr + 1), _quantized(s["x"], 0, fmt, ch))
        return dict(dx=dx, dw=dw)
    if kind == "attention":
        h = case["heads"]
        return dict(scores=_product(_quantized(s["q"], 1, fmt, groups=h), _quantized(s["k"], 1, fmt, groups=h)),
                    out=_product(_quantized(s["p"], 1, fmt, groups=h), _quantized(s["v"], 0, fmt, groups=h)))
    if kind == "gemm":
        def values(op, delta, name):
            c = op[0]
            v = (c.view(torch.int8) if name == "int8" else c.view(torch.float8_e4m3fn if name == "e4m3" else torch.float8_e5m2)).double()
            return v, delta.double().view(1, -1, 1)
        return dict(y=_product(values(s["a"], s["da"], fmt), values(s["b"], s["db"], case["fmt_b"])))
    if kind == "reference":
        return dict(y=(s["x"].double() @ s["w"].double().t()).unsqueeze(0))
    if kind == "example":
        l, r = s["l"].double(), s["r"].double()
        y = _product(_quantized(s["l"], 1, fmt, True), _quantized(s["r"], 1, fmt, True))
        ref, denom = (l @ r.t()).unsqueeze(0), (l.abs() @ r.abs().t()).unsqueeze(0)
        m = _metric(y, ref, denom)
        return dict(y=y, ref=ref, denom=denom, sums=m[0:6], backward=m[8:16])
    if kind == "stats":
        v, per_row, delta = _quantized(s["x"], 1, fmt, case["channel"])
        values = (v * per_row)[0]
        x = s["x"].double().reshape(-1)
        mean = x.mean()
        c = x - mean
        z = torch.zeros((), dtype=torch.float64, device=DEV)
        moments = torch.stack([z + x.numel(), mean, c.square().mean(), (c * c * c).mean(), c.square().square().mean(), x.abs().max(), z, z])
        return dict(moments=moments, delta=delta, codes=None, values=values, metric=_metric(values.float(), s["x32"]))
    ref, out = s["x"].double() @ s["w"].double().t(), []
    for f, channel in experiments.CANDIDATES:
        name = {v: n for n, v in FMT.items()}[f]
        y = _product(_quantized(s["x"], 1, name, channel), _quantized(s["w"], 1, name, channel))[0]
        m = _metric(y, ref).cpu().numpy()
        out.append(np.concatenate([[m[0] / m[1]], m[0:6], m[12:13]]))
    return out
