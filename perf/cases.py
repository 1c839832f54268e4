"""The calls that users of this library make, at the sizes they make them: what performance work on it is
measured on.

Sizes are the GPT-3-family layer shapes of paper_2208_07339_amd/workloads.py and of the benchmark, and odd ones
of the same ranges.  A state holds what a program has in hand before the call: hidden states on the GPU, weights
that were converted when they were loaded, and the buffers a call writes into, allocated once per layer shape as
bench.py does.
"""
import torch

import paper_2208_07339_amd as L

ALPHA = 6.0       # outlier threshold of the method
CAP = 32          # capacity of the outlier list, as in the benchmark
MAX_WEIGHT = 49152 * 12288
MAX_WORK = 2048 * MAX_WEIGHT  # multiply-adds of the largest listed product


def _product(name, s, h, o, outliers, call="linear", fp16_rows=True):
    return {"name": name, "call": call, "s": s, "h": h, "o": o, "outliers": outliers, "fp16_rows": fp16_rows}


def _weight(name, h, o, quantizer):
    return {"name": name, "call": "quantize_weight", "h": h, "o": o, "quantizer": quantizer}


def listed():
    return [
        # the configuration of the smoke test: a layer so small that launches and host work are all there is
        _product("tiny", 8, 256, 512, 2),
        # one user generating token by token, weights kept as int8 only (the memory the method exists to save)
        _product("decode_1_int8_rows", 1, 5120, 20480, 7, fp16_rows=False),
        # token-by-token generation for a small batch through the widest layer: the decode benchmark
        _product("decode_16_wide", 16, 12288, 49152, 7),
        # a serving batch of generating users: too many tokens for a matrix-vector kernel, few for a GEMM
        _product("decode_96", 96, 5120, 15360, 6),
        # prompts through an attention projection
        _product("prefill_attention", 2048, 4096, 4096, 6),
        # prompts through a feed-forward layer, up: the prefill benchmark
        _product("prefill_ffn", 4096, 5120, 20480, 8),
        # prompts through the largest feed-forward layer, down: long sums, the largest call
        _product("prefill_ffn_down", 2048, 49152, 12288, 20),
        # a prompt of any length through a layer whose dimensions are multiples of nothing (pruned or merged
        # layers, output projections onto a vocabulary)
        _product("prefill_ragged", 1013, 4099, 12301, 5),
        # the asymmetric variant on one-sided hidden states (behind a ReLU-like activation)
        _product("prefill_zeropoint", 2048, 5120, 20480, 8, call="zp_linear"),
        # the method's steps called one by one, by a program that keeps the codes or shares them between layers
        _product("prefill_staged", 1024, 8192, 8192, 7, call="staged"),
        # loading a model: fp16 weights into codes and constants
        _weight("load_weight", 5120, 20480, "absmax"),
        _weight("load_weight_zeropoint", 5120, 20480, "zeropoint"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _dimension(rng, lo, hi):
    """A layer dimension: mostly multiples of 128 or 8 as layers have them, sometimes a multiple of nothing."""
    n = _log_int(rng, lo, hi)
    step = rng.choice([128, 128, 128, 8, 1])
    return max(lo, n // step * step)


def draw(rng):
    if rng.random() < 0.2:
        while True:
            h, o = _dimension(rng, 256, 49152), _dimension(rng, 512, 49152)
            if h * o <= 5120 * 20480:
                c = _weight("", h, o, rng.choice(["absmax", "zeropoint"]))
                del c["name"]
                return c
    while True:
        s = rng.choice([_log_int(rng, 1, 4096), _log_int(rng, 1, 128)])
        h, o = _dimension(rng, 256, 49152), _dimension(rng, 512, 49152)
        # products whose dimensions are not multiples of 8 do not reach the size of the largest layers
        most = MAX_WORK if h % 8 == 0 and o % 8 == 0 else 1013 * 4099 * 12301
        if h * o <= MAX_WEIGHT and s * h * o <= most:
            break
    call = rng.choice(["linear"] * 5 + ["zp_linear", "zp_linear", "staged"])
    c = _product("", s, h, o, rng.randint(0, 20), call, call != "linear" or rng.random() < 0.75)
    del c["name"]
    return c


def _hidden_states(g, s, h, outliers, one_sided):
    """N(0, 1) features, a few of which carry large one-signed values in three quarters of the tokens."""
    x = torch.empty((s, h), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    if one_sided:
        x.clamp_(min=-0.25)
    cols = torch.randperm(h, device="cuda", generator=g)[:outliers]
    n = cols.numel()
    if n:
        sign = torch.randint(0, 2, (1, n), device="cuda", generator=g) * 2.0 - 1.0
        mag = torch.rand((s, n), device="cuda", generator=g) * 50.0 + 10.0
        keep = torch.rand((s, n), device="cuda", generator=g) < 0.75
        x[:, cols] = torch.where(keep, (sign * mag).half(), x[:, cols])
    return x


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    h, o = case["h"], case["o"]
    W = torch.empty((h, o), dtype=torch.float16, device="cuda").normal_(0.0, 0.02, generator=g)
    if case["call"] == "quantize_weight":
        return {"call": case["call"], "quantizer": case["quantizer"], "W": W,
                "ws": L.Workspace.allocate(1, h, o, 1)}
    s, zp = case["s"], case["call"] == "zp_linear"
    X = _hidden_states(g, s, h, case["outliers"], zp)
    ws = L.Workspace.allocate(s, h, o, CAP)
    qw = L.zp_quantize_weight(W, ws) if zp else L.quantize_weight(W, ws)
    if not case["fp16_rows"]:
        qw.W = None
    outl = L.Outliers(torch.zeros(CAP, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"),
                      torch.zeros(1, dtype=torch.int32, device="cuda"), CAP)
    Xq = torch.zeros(L.xq_bytes(s, h), dtype=torch.int8, device="cuda")
    Xo = torch.zeros((s, L.opad(CAP)), dtype=torch.float16, device="cuda")
    if zp:
        rows = L.ZpRows(Xq, torch.zeros((s, 4), dtype=torch.int32, device="cuda"), Xo, s, h)
    else:
        rows = L.QuantizedRows(Xq, torch.zeros(s, dtype=torch.float16, device="cuda"), Xo, s, h)
    out = torch.zeros((s, o), dtype=torch.float16, device="cuda")
    return {"call": case["call"], "X": X, "qw": qw, "outl": outl, "rows": rows, "ws": ws, "out": out}


def run(state):
    if state["call"] == "quantize_weight":
        if state["quantizer"] == "zeropoint":
            qw = L.zp_quantize_weight(state["W"], state["ws"])
            return {"codes": qw.Wq, "constants": qw.zc}
        qw = L.quantize_weight(state["W"], state["ws"])
        return {"codes": qw.Wq, "constants": qw.cw}
    X, qw, outl, rows, ws, out = (state[k] for k in ("X", "qw", "outl", "rows", "ws", "out"))
    if state["call"] == "zp_linear":
        L.zp_linear(X, qw, ALPHA, outl, rows, ws, out)
        constants = rows.zc
    elif state["call"] == "staged":
        L.find_outliers(X, ALPHA, CAP, ws, outl)
        L.quantize_rows(X, outl, rows)
        L.matmul(rows, outl, qw, ws, out)
        constants = rows.cx
    else:
        L.linear(X, qw, ALPHA, outl, rows, ws, out)
        constants = rows.cx
    return {"out": out, "codes": rows.Xq, "constants": constants, "outlier_values": rows.Xo, "count": outl.count,
            "status": outl.status}


def work(case):
    h, o = case["h"], case["o"]
    if case["call"] == "quantize_weight":  # fp16 weights in; codes and constants out
        return {"bytes": 3 * h * o + (16 if case["quantizer"] == "zeropoint" else 2) * o, "flops": 4 * h * o}
    s, n = case["s"], case["outliers"]
    record = 16 if case["call"] == "zp_linear" else 2  # constants of a row or column
    # X, the codes and constants of W, the outlier rows of W (fp16, or among the codes); the codes and constants
    # of X, the outlier columns, the result
    read = 2 * s * h + h * o + record * o + (2 * n * o if case["fp16_rows"] else 0)
    written = s * h + record * s + 2 * s * n + 2 * s * o
    return {"bytes": read + written, "flops": 2 * s * h * o + 2 * s * n * o}


def tolerance(case):
    if case["call"] == "quantize_weight":
        return "exact"
    # Against the same product in 64 bits, rounded once to fp16: rel 5e-6, max 1e-3 (a value next to a tie rounds
    # the other way: one fp16 step, in 2 of 10 000 outputs).  Four times that; one such value among the 512
    # outputs of the smallest call is up to 5e-5 of the whole, hence rel 1e-4 and not 2e-5.
    return {"rel": 1e-4, "max": 2e-3}
