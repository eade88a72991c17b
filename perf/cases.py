"""The work this library is timed on: its public calls over the sizes, data
types and operand contracts that programs give them.

A case is a dict of plain values.  `op` names the operation, `call` how a
program reaches it: "exec" is a persistent executor, planned once and run on
every new input; "once" the one-shot call, which returns a new output tensor.

  gemm_i16   packed INT16 GEMM, int32 sums; `bound` is the promised largest
             |x| (0: none): 127 int8 products, 256 and 2048 exact 16-bit
             float products, 8000 three int8 products, 0 four of them
  gemm_s24   INT32 GEMM under the smul24 contract (full signed 24-bit values)
  conv       convolution, `dt` i16 / f32 / i32 (smul24)
  attn       attention core (Q K^T) V, `dt` f32 / i32
  sdpa       multi-head softmax attention, float32, plain or causal
  lenet      the LeNet-5-shaped INT32 pipeline

Pooling and min/max are left out: each is one pass over memory.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2606_09905_amd import qx


def listed():
    return [
        # one small INT16 product: an inner step of a host program, bound by its launch
        dict(name="gemm_i16_256", op="gemm_i16", call="exec", batch=1, M=256, N=256, K=256, bound=1024),
        # INT16 data with no range promise (sensor or audio samples) and ragged sizes, through the one-shot call
        dict(name="gemm_i16_ragged_full", op="gemm_i16", call="once", batch=1, M=1000, N=777, K=1501, bound=0),
        # the largest single INT16 product
        dict(name="gemm_i16_8192", op="gemm_i16", call="exec", batch=1, M=8192, N=8192, K=8192, bound=256),
        # a large batch of INT16 products
        dict(name="gemm_i16_64x2048", op="gemm_i16", call="exec", batch=64, M=2048, N=2048, K=2048, bound=256),
        # one INT32 product of ordinary size
        dict(name="gemm_s24_1024", op="gemm_s24", call="exec", batch=1, M=1024, N=1024, K=1024),
        # a batch of INT32 products
        dict(name="gemm_s24_16x512", op="gemm_s24", call="exec", batch=16, M=512, N=512, K=512),
        # a 3x3 layer of a residual network, quantised and float
        dict(name="conv_i16_56", op="conv", call="exec", dt="i16", N=8, Ci=64, H=56, W=56, Co=128, KH=3, KW=3,
             stride=1, pad=1, bound=256),
        dict(name="conv_f32_56", op="conv", call="exec", dt="f32", N=8, Ci=64, H=56, W=56, Co=128, KH=3, KW=3,
             stride=1, pad=1, bound=0),
        # the attention core over a long sequence, float and integer
        dict(name="attn_f32_4096", op="attn", call="exec", dt="f32", L=4096, d=64, bound=0),
        dict(name="attn_i32_4096", op="attn", call="exec", dt="i32", L=4096, d=64, bound=64),
        # causal self-attention of a prompt, 32 heads
        dict(name="sdpa_causal_32x4096", op="sdpa", call="exec", BH=32, L=4096, d=64, scale=1.0, causal=True),
        # a whole small integer network on a batch of images
        dict(name="lenet_4096", op="lenet", call="exec", B=4096),
    ]


def _log(rng, lo, hi):
    """An integer from [lo, hi], even over its logarithm; half of them odd or ragged."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if v >= 32 and rng.random() < 0.5:
        v = v // 16 * 16
    return max(lo, min(hi, v))


def draw(rng):
    op = rng.choice(["gemm_i16", "gemm_i16", "gemm_s24", "gemm_s24", "conv", "conv", "attn", "attn", "sdpa", "lenet"])
    call = rng.choice(["exec", "exec", "once"])
    if op in ("gemm_i16", "gemm_s24"):
        while True:
            batch = rng.choice([1, 1, _log(rng, 2, 64)])
            M, N, K = (_log(rng, 16, 8192) for _ in range(3))
            bound = rng.choice([127, 256, 1024, 2048, 8000, 0]) if op == "gemm_i16" else 0
            # INT32 operands and wide INT16 ones cost several products each
            cap = 2.0 ** 38 if op == "gemm_i16" and 0 < bound <= 2048 else 2.0 ** 34
            if batch * M * N * K <= cap and batch * (M * K + K * N + M * N) <= 2 ** 28:
                break
        c = dict(op=op, call=call, batch=batch, M=M, N=N, K=K)
        if op == "gemm_i16":
            c["bound"] = bound
        return c
    if op == "conv":
        while True:
            k = rng.choice([1, 3, 3, 3, 5])
            c = dict(op=op, call=call, dt=rng.choice(["i16", "f32", "i32"]), N=_log(rng, 1, 32),
                     Ci=rng.choice([3, 16, 32, 64, 64, 128, 256]), H=_log(rng, 7, 112), W=_log(rng, 7, 112),
                     Co=rng.choice([16, 33, 64, 128, 256]), KH=k, KW=k, stride=rng.choice([1, 1, 2]), pad=k // 2)
            if work_of_conv(c) <= 2.0 ** 34:
                break
        c["bound"] = rng.choice([127, 256, 1024, 0]) if c["dt"] == "i16" else 0
        return c
    if op == "attn":
        while True:
            c = dict(op=op, call=call, dt=rng.choice(["f32", "i32"]), L=_log(rng, 64, 8192),
                     d=rng.choice([32, 64, 64, 96, 128]))
            if c["L"] * c["L"] * c["d"] <= 2.0 ** 32:
                break
        c["bound"] = rng.choice([64, 127]) if c["dt"] == "i32" else 0
        return c
    if op == "sdpa":
        while True:
            d = rng.choice([32, 64, 64, 80, 128])
            c = dict(op=op, call=call, BH=_log(rng, 1, 128), L=_log(rng, 64, 8192), d=d,
                     scale=rng.choice([1.0, d ** -0.5]), causal=rng.random() < 0.5)
            if c["BH"] * c["L"] * c["L"] * d <= 2.0 ** 34:
                break
        return c
    return dict(op="lenet", call="exec", B=_log(rng, 1, 8192))


def work_of_conv(c):
    """Multiply-adds of a convolution."""
    ho, wo = qx.conv_out_hw(c["H"], c["W"], c["KH"], c["KW"], c["stride"], c["pad"])
    return float(c["N"] * c["Co"] * ho * wo) * c["Ci"] * c["KH"] * c["KW"]


def _inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def ints(shape, lo, hi, dtype):
        return torch.randint(lo, hi + 1, shape, generator=g, device="cuda", dtype=dtype)

    def normal(shape, scale):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale

    op = c["op"]
    if op == "gemm_i16":
        b = c["bound"]
        lo, hi = (-b, b - 1 if b != 127 else b) if b else (-32768, 32767)
        return [ints((c["batch"], c["M"], c["K"]), lo, hi, torch.int16),
                ints((c["batch"], c["K"], c["N"]), lo, hi, torch.int16)]
    if op == "gemm_s24":
        lo, hi = -(1 << 23), (1 << 23) - 1
        return [ints((c["batch"], c["M"], c["K"]), lo, hi, torch.int32),
                ints((c["batch"], c["K"], c["N"]), lo, hi, torch.int32)]
    if op == "conv":
        xs, ws = (c["N"], c["Ci"], c["H"], c["W"]), (c["Co"], c["Ci"], c["KH"], c["KW"])
        if c["dt"] == "f32":
            return [normal(xs, 1.0), normal(ws, (c["Ci"] * c["KH"] * c["KW"]) ** -0.5)]
        if c["dt"] == "i32":
            lo, hi, dt = -(1 << 23), (1 << 23) - 1, torch.int32
        else:
            b, dt = c["bound"], torch.int16
            lo, hi = (-b, b - 1 if b != 127 else b) if b else (-32768, 32767)
        return [ints(xs, lo, hi, dt), ints(ws, lo, hi, dt)]
    if op == "attn":
        if c["dt"] == "f32":
            return [normal((c["L"], c["d"]), c["d"] ** -0.5) for _ in range(3)]
        b = c["bound"]
        return [ints((c["L"], c["d"]), -b, b - 1 if b != 127 else b, torch.int32) for _ in range(3)]
    if op == "sdpa":
        # scores of unit variance at scale 1, of d^(1/2) times that otherwise scaled back
        s = c["d"] ** -0.25 if c["scale"] == 1.0 else 1.0
        return [normal((c["BH"], c["L"], c["d"]), s) for _ in range(3)]
    x = ints((c["B"], 1, 32, 32), 0, 255, torch.int32)
    shapes = ((6, 1, 5, 5), (16, 6, 5, 5), (400, 120), (120, 84), (84, 10))
    return [x] + [ints(s, -3, 3, torch.int32) for s in shapes]


def _executor(c):
    op = c["op"]
    if op == "gemm_i16":
        return qx.Executor.gemm_i16i32(c["M"], c["N"], c["K"], c["batch"], c["bound"], c["bound"])
    if op == "gemm_s24":
        return qx.Executor.gemm_i32_s24(c["M"], c["N"], c["K"], c["batch"])
    if op == "conv":
        dims = [c[k] for k in ("N", "Ci", "H", "W", "Co", "KH", "KW", "stride", "pad")]
        if c["dt"] == "i16":
            return qx.Executor.conv2d(*dims, c["bound"], c["bound"])
        return qx.Executor.conv2d_t(c["dt"], *dims)
    if op == "attn":
        return qx.Executor.attn(c["dt"], c["L"], c["d"], c["bound"])
    if op == "sdpa":
        return qx.Executor.sdpa_f32(c["BH"], c["L"], c["d"], c["scale"], c["causal"])
    return qx.Executor.lenet_i32(c["B"])


def prepare(case, seed):
    state = dict(case=case, inputs=_inputs(case, seed))
    if case["call"] == "exec":
        ex = _executor(case)
        state["exec"] = ex
        state["out"] = torch.empty(ex.out_shape, dtype=ex.out_dtype, device="cuda")
    return state


def run(state):
    c, x = state["case"], state["inputs"]
    if c["call"] == "exec":
        return state["exec"].run(x, state["out"])
    op = c["op"]
    if op == "gemm_i16":
        return qx.qgemm_i16i32(x[0], x[1], c["bound"], c["bound"])
    if op == "gemm_s24":
        return qx.qgemm_i32_s24(x[0], x[1])
    if op == "conv":
        if c["dt"] == "i16":
            return qx.conv2d_gemm(x[0], x[1], c["stride"], c["pad"], c["bound"], c["bound"])
        return qx.conv2d_gemm_t(x[0], x[1], c["stride"], c["pad"])
    if op == "attn":
        return qx.attn_core(*x, c["bound"])
    return qx.sdpa_f32(*x, c["scale"], c["causal"])


def work(case):
    c, op = case, case["op"]
    if op in ("gemm_i16", "gemm_s24"):
        e = 2 if op == "gemm_i16" else 4
        b, M, N, K = c["batch"], c["M"], c["N"], c["K"]
        return {"bytes": float(b * (e * (M * K + K * N) + 4 * M * N)), "flops": 2.0 * b * M * N * K}
    if op == "conv":
        e = 2 if c["dt"] == "i16" else 4
        ho, wo = qx.conv_out_hw(c["H"], c["W"], c["KH"], c["KW"], c["stride"], c["pad"])
        return {"bytes": float(e * (c["N"] * c["Ci"] * c["H"] * c["W"] + c["Co"] * c["Ci"] * c["KH"] * c["KW"])
                               + 4 * c["N"] * c["Co"] * ho * wo), "flops": 2.0 * work_of_conv(c)}
    if op == "attn":
        return {"bytes": 16.0 * c["L"] * c["d"], "flops": 4.0 * c["L"] * c["L"] * c["d"]}
    if op == "sdpa":
        pairs = c["L"] * (c["L"] + 1) / 2 if c["causal"] else c["L"] * c["L"]
        return {"bytes": 16.0 * c["BH"] * c["L"] * c["d"], "flops": 4.0 * c["BH"] * pairs * c["d"]}
    weights = 6 * 25 + 16 * 150 + 400 * 120 + 120 * 84 + 84 * 10
    macs = 6 * 28 * 28 * 25 + 16 * 10 * 10 * 150 + 400 * 120 + 120 * 84 + 84 * 10
    return {"bytes": 4.0 * (c["B"] * (1024 + 10) + weights), "flops": 2.0 * c["B"] * macs}


def tolerance(case):
    # integers are exact mod 2^32; float32 sums differ by their order: against
    # float64, 8.3e-7 and 9.1e-6 were the largest seen over these ranges
    if case["op"] == "sdpa" or case.get("dt") == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return "exact"


def _wrap(v):
    """Whole numbers held in float64 or int64 as int32, mod 2^32."""
    v = v.to(torch.int64) & 0xFFFFFFFF
    return torch.where(v >= 1 << 31, v - (1 << 32), v).to(torch.int32)


def _sext24(x):
    v = x.to(torch.int64) & 0xFFFFFF
    return torch.where(v >= 1 << 23, v - (1 << 24), v)


def _dot(a, b):
    """a @ b of int64 matrices with |a| < 2^24, |b| < 2^24, mod 2^32: a in two
    halves of 12 bits, so that every float64 partial sum is a whole number
    below 2^53 (up to 2^17 terms)."""
    hi = a >> 12
    lo = a - (hi << 12)
    bd = b.double()
    h = (hi.double() @ bd).to(torch.int64)
    return _wrap((h << 12) + (lo.double() @ bd).to(torch.int64))


def _columns(x, KH, KW, stride, pad):
    """im2col of float64 [Ci][H][W] -> [Ci KH KW][Ho Wo]."""
    return F.unfold(x[None], (KH, KW), padding=pad, stride=stride)[0]


def exact(case, seed):
    c, x = case, _inputs(case, seed)
    op = c["op"]
    if op == "gemm_i16":
        return torch.stack([_wrap(a.double() @ b.double()) for a, b in zip(*x)])
    if op == "gemm_s24":
        return torch.stack([_dot(_sext24(a), _sext24(b)) for a, b in zip(*x)])
    if op == "conv":
        ho, wo = qx.conv_out_hw(c["H"], c["W"], c["KH"], c["KW"], c["stride"], c["pad"])
        w = x[1].reshape(c["Co"], -1)
        out = []
        for img in x[0]:
            col = _columns(img.double(), c["KH"], c["KW"], c["stride"], c["pad"])
            if c["dt"] == "f32":
                y = w.double() @ col
            elif c["dt"] == "i32":
                y = _dot(w.to(torch.int64), col.to(torch.int64))
            else:
                y = _wrap(w.double() @ col)
            out.append(y.reshape(c["Co"], ho, wo))
        return torch.stack(out)
    if op == "attn":
        q, k, v = (t.double() for t in x)
        s = q @ k.t().contiguous()
        return s @ v if c["dt"] == "f32" else _wrap(s @ v)
    if op == "sdpa":
        out = torch.empty(x[0].shape, dtype=torch.float64, device="cuda")
        for b in range(c["BH"]):
            q, k, v = (t[b].double() for t in x)
            s = (q @ k.t().contiguous()) * c["scale"]
            if c["causal"]:
                s.masked_fill_(torch.ones_like(s, dtype=torch.bool).triu_(1), -math.inf)
            out[b] = torch.softmax(s, dim=-1) @ v
        return out
    h, w1, w2, f1, f2, f3 = x

    def conv_pool(h, w, ho):
        cols = torch.stack([_columns(i.double(), 5, 5, 1, 0) for i in h]).to(torch.int64)
        y = _dot(_sext24(w).reshape(w.shape[0], -1), cols.transpose(0, 1).reshape(cols.shape[1], -1))
        y = y.reshape(w.shape[0], len(h), ho, ho).transpose(0, 1).clamp_min(0).to(torch.int64)
        y = y[:, :, 0::2, 0::2] + y[:, :, 0::2, 1::2] + y[:, :, 1::2, 0::2] + y[:, :, 1::2, 1::2]
        return _sext24(y >> 2)

    h = conv_pool(conv_pool(_sext24(h), w1, 28), w2, 10).reshape(c["B"], 400)
    h = _sext24(_dot(h, _sext24(f1)).clamp_min(0))
    h = _sext24(_dot(h, _sext24(f2)).clamp_min(0))
    return _dot(h, _sext24(f3))
