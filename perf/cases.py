"""Workloads of libquake as a user's program calls them, with sizes, inputs and
64-bit results: row softmax (scores, masked scores, vocabulary rows), the GELU
and SiLU of an MLP's activations, the MLP's two linear layers, and attention.

A case is a dict of plain values with a "kind":

  elementwise  op ("gelu", "silu", "sigmoid", "exp"), n, dtype, mode
  softmax      rows, cols, dtype, mode, t; workspace: the program keeps the
               zero-filled workspace of quake_softmax_ws for this shape
  causal       rows, cols (one square score block per `cols` rows), dtype, mode, t
  linear       m, n, k, dtype, mode, gelu (False: the product alone)
  attention    heads, seq, dtype, mode, causal

`prepare` makes what such a program holds before the call, `run` is one call
through the public entry points, `exact` the same operator in 64-bit torch with
QuAKE's exponential taken as the real function of Eq. 2 and Eq. 6 (2^i times the
polynomial of the fraction), so it has no rounding of its own.
"""
from __future__ import annotations

import math

import torch

from paper_2412_00408_amd import quake as q

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}
LN2 = math.log(2.0)
GELU_A = 1.0 / 0.044715
GELU_K = 2.0 * 0.044715 * math.sqrt(2.0 / math.pi)
BIAS = 0.0436                       # first-order QuAKE outside softmax


def listed() -> list[dict]:
    return [
        # the smallest call: a classifier's or router's scores for one batch; launch latency
        dict(name="softmax_f32_64x128", kind="softmax", rows=64, cols=128, dtype="f32",
             mode="quake2", t=1.0, workspace=False),
        # the activation of a BERT-base MLP over 4096 tokens
        dict(name="gelu_bf16_4096x3072", kind="elementwise", op="gelu", n=4096 * 3072,
             dtype="bf16", mode="quake2"),
        # the largest elementwise call: a gated MLP's SiLU over a long prefill batch
        dict(name="silu_f16_2p28", kind="elementwise", op="silu", n=1 << 28, dtype="f16",
             mode="quake2"),
        # next-token probabilities over a 128256-word vocabulary: one decode step of a batch of 64
        dict(name="lmhead_f32_64x128256", kind="softmax", rows=64, cols=128256, dtype="f32",
             mode="quake2", t=1.0, workspace=True),
        # materialised causal attention scores of a ragged length (8 x 12 heads of 1001 tokens)
        dict(name="causal_bf16_96x1001", kind="causal", rows=96 * 1001, cols=1001, dtype="bf16",
             mode="quake2", t=0.125),
        # BERT-base MLP up-projection with its GELU, 4096 tokens
        dict(name="linear_gelu_bf16_4096x3072x768", kind="linear", m=4096, n=3072, k=768,
             dtype="bf16", mode="quake2", gelu=True),
        # BERT-base MLP down-projection, 4096 tokens: a long k and few output columns
        dict(name="linear_bf16_4096x768x3072", kind="linear", m=4096, n=768, k=3072,
             dtype="bf16", mode="quake2", gelu=False),
        # the up-projection of a larger model over a prefill batch: the largest product
        dict(name="linear_gelu_f16_16384x4096x1024", kind="linear", m=16384, n=4096, k=1024,
             dtype="f16", mode="exact", gelu=True),
        # the up-projection for a few tokens (a decode step of 37 sequences): the weight's bytes
        dict(name="linear_gelu_f16_37x3072x768", kind="linear", m=37, n=3072, k=768,
             dtype="f16", mode="quake2", gelu=True),
        # causal self-attention of 8 x 12 heads over 512 tokens
        dict(name="attention_bf16_96x512_causal", kind="attention", heads=96, seq=512,
             dtype="bf16", mode="quake2", causal=True),
        # an encoder's attention (no mask) over 2048 tokens
        dict(name="attention_bf16_32x2048", kind="attention", heads=32, seq=2048,
             dtype="bf16", mode="quake2", causal=False),
        # causal prefill of a ragged length past 2048 tokens
        dict(name="attention_f16_16x4001_causal", kind="attention", heads=16, seq=4001,
             dtype="f16", mode="quake2", causal=True),
    ]


def _log(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case: dict) -> float:
    w = work(case)
    return w["bytes"] / 8e12 + w["flops"] / 2.5e15


def draw(rng) -> dict:
    mode = rng.choice(["quake2"] * 5 + ["exact", "quake1", "quake2m"])
    half = rng.choice(["bf16", "f16"])
    any_dtype = rng.choice(["bf16", "f16", "f32"])
    largest = max(_cost(c) for c in listed())
    kind = rng.choice(["elementwise", "softmax", "causal", "linear", "linear", "attention",
                       "attention"])
    while True:
        if kind == "elementwise":
            case = dict(kind=kind, op=rng.choice(["gelu", "silu", "sigmoid", "exp"]),
                        n=_log(rng, 4096, 1 << 28), dtype=any_dtype, mode=mode)
        elif kind == "softmax":
            cols = _log(rng, 64, 131072)
            case = dict(kind=kind, rows=_log(rng, 16, max(32, (1 << 26) // cols)), cols=cols,
                        dtype=any_dtype, mode=mode, t=rng.choice([1.0, 0.7]),
                        workspace=cols > 16384)
        elif kind == "causal":
            seq = _log(rng, 64, 4096)
            case = dict(kind=kind, rows=seq * rng.randint(1, max(1, min(96, (1 << 26) // (seq * seq)))),
                        cols=seq, dtype=any_dtype, mode=mode, t=0.125)
        elif kind == "linear":
            case = dict(kind=kind, m=_log(rng, 1, 16384), n=_log(rng, 256, 4096),
                        k=8 * _log(rng, 8, 512), dtype=half, mode=mode, gelu=rng.random() < 0.7)
        else:
            case = dict(kind=kind, heads=rng.choice([8, 12, 16, 32, 40, 64, 96]),
                        seq=_log(rng, 64, 8192), dtype=half, mode=mode,
                        causal=rng.random() < 0.6)
        if _cost(case) <= largest:
            return case


# ---------------------------------------------------------------- inputs

def _gen(seed: int) -> torch.Generator:
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(shape, std, dtype, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _inputs(case: dict, seed: int) -> dict:
    g = _gen(seed)
    dt = DTYPES[case["dtype"]]
    kind = case["kind"]
    if kind == "elementwise":
        n = case["n"]
        if case["op"] in ("gelu", "exp"):
            return dict(x=_normal(n, 1.5, dt, g))                   # pre-activations
        x = torch.rand(n, generator=g, device="cuda", dtype=torch.float32).mul_(24.0).sub_(12.0)
        far = torch.randint(n, (n // 100,), generator=g, device="cuda")   # 1 % saturated gates
        x[far] = 80.0 * torch.sign(x[far])
        return dict(x=x.to(dt))
    if kind == "softmax":
        x = torch.randn((case["rows"], case["cols"]), generator=g, device="cuda").mul_(3.0)
        if case["cols"] > 16384:                                    # a few likely words per row
            top = torch.randint(case["cols"], (case["rows"], 16), generator=g, device="cuda")
            x.scatter_(1, top, 20.0)
        return dict(x=x.to(dt))
    if kind == "causal":                                            # q k^T of unit-variance heads
        return dict(x=_normal((case["rows"], case["cols"]), 8.0, dt, g))
    if kind == "linear":
        return dict(x=_normal((case["m"], case["k"]), 1.0, dt, g),
                    w=_normal((case["n"], case["k"]), 1.5 / math.sqrt(case["k"]), dt, g))
    h, s = case["heads"], case["seq"]
    # v^T rows padded to 8 elements, the layout of a key/value cache
    vt = _normal((h, 64, (s + 7) // 8 * 8), 1.0, dt, g)
    return dict(q=_normal((h, s, 64), 1.0, dt, g), k=_normal((h, s, 64), 1.0, dt, g), vt=vt)


def prepare(case: dict, seed: int) -> dict:
    st = dict(case=case, **_inputs(case, seed))
    if case["kind"] == "attention":
        st["vt"] = st["vt"][:, :, :case["seq"]]
    if case["kind"] == "softmax":
        st["workspace"] = (q.softmax_workspace(case["rows"], case["cols"], st["x"].dtype,
                                               st["x"].device) if case["workspace"] else None)
    return st


def run(st: dict):
    c = st["case"]
    kind, mode = c["kind"], c["mode"]
    if kind == "elementwise":
        if c["op"] == "gelu":
            return q.quake_gelu(st["x"], mode=mode)
        if c["op"] == "exp":
            return q.quake_exp(st["x"], mode=mode)
        return q.quake_sigmoid(st["x"], mode=mode, silu=c["op"] == "silu")
    if kind == "softmax":
        return q.quake_softmax(st["x"], mode=mode, t=c["t"], workspace=st["workspace"])
    if kind == "causal":
        return q.quake_softmax_causal(st["x"], mode=mode, t=c["t"])
    if kind == "linear":
        return q.quake_linear_gelu(st["x"], st["w"], mode=mode, gelu=c["gelu"])
    return q.quake_attention(st["q"], st["k"], st["vt"], mode=mode, causal=c["causal"])


# ---------------------------------------------------------------- what a pass cannot do without

def work(case: dict) -> dict:
    e = BYTES[case["dtype"]]
    kind = case["kind"]
    if kind == "elementwise":                      # each element once in, once out
        return dict(bytes=2 * e * case["n"], flops=8 * case["n"])
    if kind == "softmax":
        n = case["rows"] * case["cols"]
        return dict(bytes=2 * e * n, flops=8 * n)
    if kind == "causal":                           # the live half in, the whole block out
        live = case["rows"] // case["cols"] * (case["cols"] * (case["cols"] + 1) // 2)
        return dict(bytes=e * (live + case["rows"] * case["cols"]), flops=8 * live)
    if kind == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(bytes=e * (m * k + n * k + m * n), flops=2 * m * n * k)
    h, s = case["heads"], case["seq"]
    pairs = s * (s + 1) // 2 if case["causal"] else s * s
    return dict(bytes=4 * e * h * s * 64, flops=4 * 64 * h * pairs)


def tolerance(case: dict) -> dict:
    """About four times the distance to `exact` measured over the ranges of
    `draw`: one rounding to the output format (1.7e-3 in bfloat16, 2.2e-4 in
    binary16; largest 3.9e-3 and 4.9e-4), in binary32 the 2^-17 spacing of the
    exponential's argument (softmax 1.6e-6, largest 5e-6); attention also rounds
    its probabilities (2.3e-3 and 2.9e-4; largest 1.9e-2 and 3.4e-3)."""
    if case["dtype"] == "f32":
        return dict(rel=2e-5 if case.get("op") == "exp" else 6e-6, max=2e-5)
    if case["kind"] == "attention":
        return (dict(rel=9e-3, max=8e-2) if case["dtype"] == "bf16" else dict(rel=1.2e-3, max=1.4e-2))
    return dict(rel=7e-3, max=1.6e-2) if case["dtype"] == "bf16" else dict(rel=9e-4, max=2e-3)


# ---------------------------------------------------------------- the same in 64 bits

def _q(v: torch.Tensor, mode: str) -> torch.Tensor:
    """2^v with the exponential of `mode`, v in float64 (base-2 exponent)."""
    if mode == "exact":
        return torch.exp2(v)
    v = v.clamp(-1000.0, 1000.0)
    i = torch.floor(v)
    a = 1.0 + (v - i)
    if mode == "quake2":
        a = (a * a + 2.0) / 3.0
    elif mode == "quake2m":
        a = torch.where(a == 1.0, a, (0.337189435 * a - 0.0167425927) * a + 0.681277931)
    return torch.exp2(i).mul_(a)


def _bias(mode: str) -> float:
    return BIAS if mode == "quake1" else 0.0


def _pointwise(x: torch.Tensor, op: str, mode: str) -> torch.Tensor:
    x = x.double()
    if op == "exp":
        return _q(x / LN2 - _bias(mode), mode)
    if op == "gelu":
        return x / (1.0 + _q(-GELU_K / LN2 * x * (GELU_A + x * x) - _bias(mode), mode))
    e = 1.0 + _q(-x / LN2 - _bias(mode), mode)
    return x / e if op == "silu" else 1.0 / e


def _softmax_rows(x: torch.Tensor, t: float, mode: str) -> torch.Tensor:
    x = x.double()
    m = x.amax(dim=1, keepdim=True)
    p = _q((x - m) * (t / LN2), mode).masked_fill_(x == -math.inf, 0.0)
    return p / p.sum(dim=1, keepdim=True)


def exact(case: dict, seed: int):
    a = _inputs(case, seed)
    kind, mode = case["kind"], case["mode"]
    if kind == "elementwise":
        x, step = a["x"], 1 << 24
        out = torch.empty(x.shape, dtype=torch.float64, device=x.device)
        for i in range(0, x.numel(), step):
            out[i:i + step] = _pointwise(x[i:i + step], case["op"], mode)
        return out
    if kind in ("softmax", "causal"):
        x = a["x"]
        rows, cols = x.shape
        out = torch.empty(x.shape, dtype=torch.float64, device=x.device)
        step = max(1, (1 << 24) // cols)
        for r in range(0, rows, step):
            xr = x[r:r + step].double()
            if kind == "causal":
                i = torch.arange(r, r + xr.shape[0], device=x.device) % cols
                j = torch.arange(cols, device=x.device)
                xr.masked_fill_(j[None, :] > i[:, None], -math.inf)
            out[r:r + step] = _softmax_rows(xr, case["t"], mode)
        return out
    if kind == "linear":
        y = a["x"].double() @ a["w"].double().t().contiguous()
        if not case["gelu"]:
            return y
        for r in range(0, y.shape[0], 1024):
            y[r:r + 1024] = _pointwise(y[r:r + 1024], "gelu", mode)
        return y
    s = case["seq"]
    out = torch.empty(a["q"].shape, dtype=torch.float64, device="cuda")
    j = torch.arange(s, device="cuda")
    for h in range(case["heads"]):
        kt = a["k"][h].double().t().contiguous()
        v = a["vt"][h, :, :s].double().t().contiguous()
        for r in range(0, s, 2048):
            sc = a["q"][h, r:r + 2048].double() @ kt
            if case["causal"]:
                i = torch.arange(r, r + sc.shape[0], device="cuda")
                sc.masked_fill_(j[None, :] > i[:, None], -math.inf)
            out[h, r:r + 2048] = _softmax_rows(sc, 0.125, mode) @ v
    return out
