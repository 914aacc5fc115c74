"""Timed cases of the attention forward and its quantizers, with fp64 references.

Each case is one call, or one pair of calls, that a user of this library makes
through the torch binding:

* ``attention``: ``attention_mxfp4`` on Q, K, V: quantization and forward;
* ``forward``: ``forward_mxfp4`` on operands that the caller quantized before
  (a cache of MXFP4 operands, or the paper's timed scope), into a buffer that
  the caller keeps;
* ``quantize``: ``quantize_qkv`` alone;
* ``bf16``: ``forward_bf16`` on the same Q, K, V.

Inputs are seeded synthetic tensors of the repository's workloads: i.i.d.
N(0, 1), N(0, 1) with a few outlier channels of Q and K, or Student-t with four
degrees of freedom scaled to unit variance; Q, K, V in bf16 or fp32.
"""
import math

import torch

import paper_2609_04105_amd as fa

GUARD = (110, 16)   # margin and shift of the sampled guard: the paper's setting for its 1.3B video model
LOG2E = 1.4426950408889634


def _case(name, call, B, H, N, d, data="gaussian", src="bf16", out="fp32", route="plain"):
    c = dict(call=call, B=B, H=H, N=N, d=d, data=data, src=src, out=out, route=route)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call of the library: one head, one tile, fp32 inputs, quantized and attended in one call
        _case("attention_tiny", "attention", 1, 1, 128, 64, src="fp32"),
        # a short sequence on operands already quantized: launches and latency
        _case("forward_small_d64", "forward", 1, 8, 1024, 64),
        # a batch with outlier channels, the peaked rows of large-model logits
        _case("forward_outlier", "forward", 2, 16, 4096, 128, data="outlier"),
        # heavy tails at 8k, bf16 output as a model's next layer takes it
        _case("forward_student_t", "forward", 1, 32, 8192, 128, data="student_t", out="bf16"),
        # the long-sequence throughput point
        _case("forward_long", "forward", 1, 32, 16384, 128),
        # a video model's self-attention (12 heads, 7680 tokens: grids that fill no whole round), guarded, end to end
        _case("attention_video_guard", "attention", 1, 12, 7680, 128, out="bf16", route="guard"),
        # the forward of causal training with the saved row normaliser, odd sizes
        _case("attention_causal_d64", "attention", 3, 10, 1920, 64, out="bf16", route="causal_lse"),
        # FP8 probabilities and values, the accuracy control
        _case("attention_fp8_pv", "attention", 1, 24, 4096, 128, out="bf16", route="fp8"),
        # a quarter of the key pairs on the native exponential, the `accurate` policy
        _case("forward_accurate", "forward", 1, 24, 4096, 128, route="ex2_4"),
        # the bf16 forward on a shape of the paper's tables
        _case("bf16_forward", "bf16", 1, 24, 4096, 128, out="bf16"),
        # operands of the long workload
        _case("quantize_long", "quantize", 1, 32, 16384, 128),
        # fp32 activations
        _case("quantize_fp32", "quantize", 2, 16, 4096, 128, src="fp32"),
    ]


# Cost of one (query, key) pair relative to the plain MXFP4 forward, so that a drawn case stays below the largest listed.
_PAIR_COST = {"plain": 1.0, "ex2_4": 1.1, "ex2_16": 1.4, "guard": 1.1, "causal_lse": 1.0, "fp8": 1.7}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(("attention", "attention", "forward", "forward", "forward", "bf16", "quantize"))
    route = "plain"
    if call in ("attention", "forward"):
        route = rng.choice(("plain", "plain", "plain", "causal_lse", "guard", "fp8", "ex2_4", "ex2_16"))
    elif call == "quantize":
        route = rng.choice(("plain", "plain", "guard", "fp8"))
    while True:
        d = rng.choice((64, 128, 128))
        N = 128 * _log_int(rng, 1, 128)
        B = rng.choice((1, 1, 1, 2, 3, 4))
        H = _log_int(rng, 1, 48)
        pairs = B * H * N * N * (3.0 if call == "bf16" else _PAIR_COST[route])
        if B * H * N * d <= 32 * 16384 * 128 and (call == "quantize" or pairs <= 32 * 16384 ** 2):
            break
    return _case(None, call, B, H, N, d, data=rng.choice(("gaussian", "gaussian", "outlier", "student_t")),
                 src="bf16" if call == "bf16" or rng.random() < 0.7 else "fp32",
                 out=rng.choice(("fp32", "bf16")), route=route)


def _draw_qkv(case, seed):
    """Q, K, V of a case on the GPU (the recipe of the repository's workloads, drawn on the device)."""
    shape = (case["B"], case["H"], case["N"], case["d"])
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal():
        return torch.randn(shape, device="cuda", generator=g)

    def one():
        z = normal()
        if case["data"] != "student_t":
            return z
        w = torch.zeros_like(z)
        for _ in range(4):
            w += normal() ** 2
        return z / torch.sqrt(w / 4.0) / math.sqrt(2.0)

    q, k, v = one(), one(), one()
    if case["data"] == "outlier":
        ch = torch.randperm(case["d"], device="cuda", generator=g)[:math.ceil(0.02 * case["d"])]
        q[..., ch] *= 8.0
        k[..., ch] *= 8.0
    dt = _dtype(case["src"])
    return q.to(dt), k.to(dt), v.to(dt)


def _dtype(name):
    return {"fp32": torch.float32, "bf16": torch.bfloat16}[name]


def _options(route):
    return {"plain": {}, "guard": {"guard": GUARD}, "causal_lse": {"causal": True}, "fp8": {"pv_fp8": True},
            "ex2_4": {"ex2_pairs": 4}, "ex2_16": {"ex2_pairs": 16}}[route]


def prepare(case, seed):
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    q, k, v = _draw_qkv(case, seed)
    state = {"call": case["call"], "options": dict(_options(case["route"]))}
    quantized = {"anchored": case["route"] == "guard", "pv_fp8": case["route"] == "fp8"}
    if case["route"] == "causal_lse":
        state["lse"] = torch.empty((B, H, N), dtype=torch.float32, device="cuda")
    if case["call"] == "forward":
        state["operands"] = fa.quantize_qkv(q, k, v, **quantized)
        state["out"] = torch.empty((B, H, N, d), dtype=_dtype(case["out"]), device="cuda")
    else:
        state["qkv"] = (q, k, v)
        state["quantized"] = quantized
        state["out_dtype"] = _dtype(case["out"])
    return state


def run(state):
    call, lse = state["call"], state.get("lse")
    if call == "quantize":
        return fa.quantize_qkv(*state["qkv"], **state["quantized"])
    if call == "bf16":
        return fa.forward_bf16(*state["qkv"], out_dtype=state["out_dtype"])
    if call == "forward":
        out = fa.forward_mxfp4(*state["operands"], out=state["out"], lse=lse, **state["options"])
    else:
        out = fa.attention_mxfp4(*state["qkv"], out_dtype=state["out_dtype"], lse=lse, **state["options"])
    return out if lse is None else (out, lse)


def work(case):
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    values = B * H * N * d                       # of each of Q, K, V and O
    fp4, fp8 = values * (1 / 2 + 1 / 32), values * (1 + 1 / 32)
    operands = 2 * fp4 + (fp8 if case["route"] == "fp8" else fp4)
    source = 3 * values * (2 if case["src"] == "bf16" else 4)
    result = values * (2 if case["out"] == "bf16" else 4)
    if case["route"] == "causal_lse":
        result += 4 * B * H * N
        pairs = B * H * N * (N + 1) / 2
    else:
        pairs = B * H * N * N
    moved = {"attention": source + result, "forward": operands + result, "quantize": source + operands,
             "bf16": source + result}[case["call"]]
    return {"bytes": moved, "flops": 0 if case["call"] == "quantize" else 4 * pairs * d}


def tolerance(case):
    if case["call"] == "quantize":
        return "exact"                           # codes and scales are decided exactly
    if case["call"] == "bf16":
        # probabilities are rounded to bf16 before the PV product
        return {"rel": 1e-2, "max": 0.1}
    if case["out"] == "bf16":
        # another order of the fp32 sums moves values across a rounding boundary of the bf16 output
        return {"rel": 1e-3, "max": 1e-2}
    return {"rel": 1e-5, "max": 1e-3}            # fp32 sums over the keys


# ---- fp64 references (plain torch) ----

def _e2m1(a):
    """E2M1 magnitude nearest to a >= 0 (ties to the even code, saturating at 6)."""
    small = torch.round(a * 2) / 2
    mid = torch.round(a)
    big = (torch.round(a / 2) * 2).clamp(max=6.0)
    return torch.where(a < 2, small, torch.where(a < 4, mid, big))


def _mxfp4(x):
    """Represented values of blocks of 32 along the last axis: amplitude 2^floor or
    2^ceil of the block maximum, whichever has the smaller squared error (ties: ceil)."""
    v = x.double().unflatten(-1, (-1, 32))
    mant, ex = torch.frexp(v.abs().amax(-1, keepdim=True))
    ceil = torch.where(mant == 0.5, ex - 1, ex)
    floor = ex - 1

    def reps(e):
        s = torch.ldexp(torch.ones_like(mant), e)
        return torch.copysign(_e2m1(6 * v.abs() / s), v) * s / 6

    rc, rf = reps(ceil), reps(floor)
    ec, ef = ((v - rc) ** 2).sum(-1, keepdim=True), ((v - rf) ** 2).sum(-1, keepdim=True)
    return torch.where(ef < ec, rf, rc).flatten(-2)


def _e4m3(a):
    """E4M3 value nearest to 0 <= a < 464 (ties to even, subnormals kept)."""
    _, ex = torch.frexp(a)
    step = torch.ldexp(torch.ones_like(a), (ex - 1).clamp(min=-6) - 3)
    return torch.round(a / step) * step


def _mxfp8(x):
    """Represented values: the smallest power-of-two amplitude that keeps payloads <= 448."""
    v = x.double().unflatten(-1, (-1, 32))
    _, ex = torch.frexp(v.abs().amax(-1, keepdim=True))
    e = ex - 9
    s = torch.ldexp(torch.ones_like(v[..., :1]), e)
    s = torch.where(v.abs().amax(-1, keepdim=True) / s > 448, s * 2, s)
    return (torch.copysign(_e4m3(v.abs() / s), v) * s).flatten(-2)


def _directp(q, k, v, case):
    """One head's represented operator in fp64: O and the natural-log row normaliser."""
    route, N, d = case["route"], case["N"], case["d"]
    if route == "guard":                          # 128 evenly spaced anchor keys come first
        idx = torch.arange(N, device=k.device)
        anchor = idx % (N // 128) == 0
        order = torch.cat((idx[anchor], idx[~anchor]))
        k, v = k[order], v[order]
    qh, kh = _mxfp4(q), _mxfp4(k)
    vt = v.t().contiguous()
    vh = (_mxfp8(vt) if route == "fp8" else _mxfp4(vt)).t().contiguous()
    out = torch.empty((N, d), dtype=torch.float64, device=q.device)
    lse = torch.empty(N, dtype=torch.float64, device=q.device)
    step = max(128, min(N, (1 << 27) // N))
    for r0 in range(0, N, step):
        rows = slice(r0, min(r0 + step, N))
        y = (qh[rows] @ kh.t()) * (LOG2E / math.sqrt(d))
        n = y.shape[0]
        if route == "causal_lse":
            hidden = torch.arange(N, device=y.device)[None] > torch.arange(r0, r0 + n, device=y.device)[:, None]
            y = y.masked_fill(hidden, -math.inf)
        y = y.view(n, N // 32, 32)
        top = y.amax(-1, keepdim=True)
        if route == "guard":                      # the reference is fixed in fp32, step by step
            R = (y[:, :4].amax((1, 2), keepdim=True).float() + float(GUARD[0]))
            ubar = (torch.floor(top.float() - R) + 127.0).clamp(GUARD[1] + 1, 254)
            T = (R + (ubar - 127.0)).double()
            E = ubar.double() - 127.0
        else:
            E = torch.floor(top)
            T = torch.where(torch.isinf(E), torch.zeros_like(E), E)
        x = y - T + math.log2(6.0)
        if route == "fp8":
            p = _e4m3(torch.exp2(y - T + 7.0)) / 128
        else:
            p = _e2m1((1.5 * x + 1.2).clamp(min=0.0))
            if route.startswith("ex2_"):
                pair = torch.arange(32, device=y.device) // 2
                # the offset log2 6 - E is fp32 by definition (it decides scores of exactly 0, which fall on ties)
                x32 = y + (torch.tensor(math.log2(6.0), dtype=torch.float32, device=y.device) - T.float()).double()
                p = torch.where(pair % (16 // int(route[4:])) == 0, _e2m1(torch.exp2(x32)), p)
            p = p / 6
        if route == "causal_lse":
            p = p.masked_fill(torch.isinf(y), 0.0)
        M = E.amax(1, keepdim=True)
        p = (p * torch.exp2(E - M)).view(n, N)
        D = p.sum(-1, keepdim=True)
        out[rows] = (p @ vh) / D
        lse[rows] = (M.view(n) * math.log(2.0) + torch.log(D.view(n)))
    return out, lse


def exact(case, seed):
    if case["call"] == "quantize":
        return None                               # bytes: nothing but the same bytes is right
    q, k, v = _draw_qkv(case, seed)
    B, H, N, d = q.shape
    out = torch.empty((B, H, N, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, H, N), dtype=torch.float64, device="cuda")
    for b in range(B):
        for h in range(H):
            if case["call"] == "bf16":
                kd, vd = k[b, h].double(), v[b, h].double()
                step = max(128, min(N, (1 << 27) // N))
                for r0 in range(0, N, step):
                    s = (q[b, h, r0:r0 + step].double() @ kd.t()) / math.sqrt(d)
                    out[b, h, r0:r0 + step] = torch.softmax(s, -1) @ vd
            else:
                out[b, h], lse[b, h] = _directp(q[b, h], k[b, h], v[b, h], case)
    return (out, lse) if case["route"] == "causal_lse" else out
