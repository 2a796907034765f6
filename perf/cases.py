"""The performance cases of libheinsen: the calls its users make, over the range of sizes they make them at.

Every case is one call of a public scan entry point on inputs that are already on the GPU: a, b and x0 hold
what a model or a signal would, the output buffer is the caller's own.  `listed()` names the twelve kinds of
use, `draw()` gives more sizes of the same kinds, `exact()` evaluates the definition x_t = a_t x_{t-1} + b_t in
float64 with plain torch.
"""
from __future__ import annotations

import math

import torch

from paper_2311_06281_amd import binding as hs

# ---- the kinds of use ---------------------------------------------------------------------------------
#
# layout  "BND" [B, n, D] (channels contiguous) or "BDN" [B, D, n] (time contiguous)
# mode    "signed" plain numbers of any sign | "positive" promised non-negative | "logs" natural logarithms in
#         and out | "complex" signed numbers in, complex logarithm out
# data    how a, b, x0 are distributed (see _inputs)
# static  True: the entry point that never allocates

_LISTED = [
    # One time step for every channel of a batch: a recurrent model generating a token, in a serving loop.
    dict(name="decode_step", layout="BND", B=64, n=1, D=4096, mode="signed", data="gates", bf16=False, static=True),
    # One short sequence on its own: latency only.
    dict(name="single_sequence", layout="BDN", B=1, D=1, n=4096, mode="positive", data="uniform", bf16=False, static=False),
    # A layer of a linear recurrent network over a batch of prompts (training or prefill).
    dict(name="rnn_layer", layout="BND", B=8, n=4096, D=1024, mode="signed", data="gates", bf16=False, static=False),
    # The same at the largest size: long sequences, wide layer, coefficients of both signs.
    dict(name="rnn_layer_large", layout="BND", B=16, n=16384, D=2048, mode="signed", data="mixed", bf16=False, static=False),
    # The layer with its activations stored in bf16.
    dict(name="rnn_layer_bf16", layout="BND", B=8, n=8192, D=1536, mode="signed", data="gates", bf16=True, static=False),
    # Widths and lengths that are multiples of nothing, logarithms in and out (Sec. 4 of the paper as it stands).
    dict(name="ragged_layer_logs", layout="BND", B=6, n=3001, D=770, mode="logs", data="log_gates", bf16=False, static=False),
    # State-space models: a few state channels per sequence.
    dict(name="state_channels", layout="BND", B=256, n=4096, D=16, mode="signed", data="gates", bf16=False, static=False),
    # Audio or sensor tracks: very long sequences of few channels.
    dict(name="long_tracks", layout="BND", B=2, n=131072, D=96, mode="signed", data="gates", bf16=False, static=False),
    # One very long sequence (a filter over a recording, the paper's own sweep).
    dict(name="long_sequence", layout="BDN", B=1, D=1, n=1 << 26, mode="positive", data="slow", bf16=False, static=False),
    # Time-contiguous rows of gate logarithms stored in bf16, log output for the next log-domain layer.
    dict(name="log_rows_bf16", layout="BDN", B=64, D=4096, n=2048, mode="logs", data="log_gates", bf16=True, static=False),
    # Very many short windows of odd length (discounted sums over trajectories).
    dict(name="short_rows", layout="BDN", B=256, D=1024, n=100, mode="signed", data="gates", bf16=False, static=False),
    # Growing signed sequences whose values leave float32: complex logarithm out, rows of odd length.
    dict(name="complex_rows", layout="BDN", B=16, D=512, n=3001, mode="complex", data="growing", bf16=False, static=False),
]

# Ranges of B, n, D of each kind, and the most elements a drawn call has.
_RANGES = {
    "decode_step": ((1, 256), (1, 8), (256, 8192), 1 << 22),
    "single_sequence": ((1, 1), (256, 1 << 17), (1, 1), 1 << 17),
    "rnn_layer": ((1, 32), (256, 8192), (128, 4096), 1 << 26),
    "rnn_layer_large": ((4, 32), (4096, 32768), (1024, 4096), 1 << 29),
    "rnn_layer_bf16": ((1, 32), (256, 16384), (128, 4096), 1 << 28),
    "ragged_layer_logs": ((1, 16), (129, 8191), (65, 2047), 1 << 26),
    "state_channels": ((16, 1024), (512, 16384), (2, 32), 1 << 26),
    "long_tracks": ((1, 4), (1 << 15, 1 << 19), (16, 256), 1 << 26),
    "long_sequence": ((1, 1), (1 << 18, 1 << 26), (1, 1), 1 << 26),
    "log_rows_bf16": ((8, 64), (257, 4096), (256, 4096), 1 << 29),
    "short_rows": ((16, 512), (8, 256), (64, 2048), 1 << 26),
    "complex_rows": ((1, 32), (1000, 8192), (64, 2048), 1 << 26),
}
_EVEN = {"log_rows_bf16", "rnn_layer_bf16", "rnn_layer_large", "rnn_layer"}  # sizes are usually chosen round there


def listed():
    return [dict(c) for c in _LISTED]


def draw(rng):
    """One more call of one of the kinds: sizes log-uniform over the kind's range, round ones and odd ones."""
    case = dict(rng.choice(_LISTED))
    kind = case.pop("name")
    (b, n, d, most) = _RANGES[kind]
    while True:
        def size(lo_hi, unit):
            lo, hi = lo_hi
            v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
            if unit > 1 and v > unit:
                v = v // unit * unit
            return min(max(v, lo), hi)

        unit = 64 if rng.random() < (0.7 if kind in _EVEN else 0.3) else 1
        case["B"], case["n"], case["D"] = size(b, 1), size(n, unit), size(d, unit)
        if case["B"] * case["n"] * case["D"] <= most:
            return case


# ---- one case ---------------------------------------------------------------------------------------------

_FLAGS = {
    "signed": 0,
    "positive": hs.HEINSEN_POSITIVE | hs.HEINSEN_X0_SCALAR,
    "logs": hs.HEINSEN_LOG_INPUTS | hs.HEINSEN_LOG_OUTPUT,
    "complex": hs.HEINSEN_LOG_OUTPUT | hs.HEINSEN_OUT_COMPLEX,
}


def _inputs(case, seed):
    """a, b, x0 on the GPU as the caller stores them."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, n, D = case["B"], case["n"], case["D"]
    shape = (B, n, D) if case["layout"] == "BND" else (B, D, n)

    def normal(mean, std, size=shape):
        return torch.empty(size, dtype=torch.float32, device="cuda").normal_(mean, std, generator=g)

    def uniform(lo, hi, size=shape):
        return torch.empty(size, dtype=torch.float32, device="cuda").uniform_(lo, hi, generator=g)

    data = case["data"]
    if data == "uniform":       # decay anywhere between a half and one, positive input, one start value
        a, b, x0 = uniform(0.5, 1.0), uniform(0.0, 1.0), torch.ones(1, dtype=torch.float32, device="cuda")
    elif data == "slow":        # decay within 1e-4 of one
        a, b = normal(-1e-7, 1e-4).exp_(), uniform(0.0, 1e-3)
        x0 = torch.ones(1, dtype=torch.float32, device="cuda")
    elif data == "gates":       # sigmoid gates, signed input
        a, b, x0 = normal(2.0, 1.0).sigmoid_(), normal(0.0, 1.0), normal(0.0, 1.0, (B * D,))
    elif data == "mixed":       # coefficients of both signs
        a, b, x0 = uniform(-1.0, 1.0), normal(0.0, 1.0), normal(0.0, 1.0, (B * D,))
    elif data == "log_gates":   # logarithms of sigmoid gates, of positive inputs and of x_0 = 1
        a, b = torch.nn.functional.logsigmoid(normal(0.0, 1.0)), normal(-1.0, 1.0)
        x0 = torch.zeros(B * D, dtype=torch.float32, device="cuda")
    elif data == "growing":     # coefficients of both signs, on average above one in magnitude
        a = normal(0.02, 0.3).exp_().mul_(uniform(-1.0, 1.0).sign_())
        b, x0 = normal(0.0, 1.0), normal(0.0, 1.0, (B * D,))
    else:
        raise ValueError(data)
    if case["bf16"]:
        a, b = a.to(torch.bfloat16), b.to(torch.bfloat16)
    return a, b, x0


def prepare(case, seed):
    a, b, x0 = _inputs(case, seed)
    shape = tuple(a.shape) + ((2,) if case["mode"] == "complex" else ())
    flags = _FLAGS[case["mode"]] | (hs.HEINSEN_IN_BF16 if case["bf16"] else 0)
    return {
        "a": a, "b": b, "x0": x0, "out": torch.empty(shape, dtype=torch.float32, device="cuda"),
        "B": case["B"], "D": case["D"], "n": case["n"], "layout": hs.LAYOUTS[case["layout"]], "flags": flags,
        "call": hs.heinsen_scan_static if case["static"] else hs.heinsen_scan,
    }


def run(state):
    s = state
    s["call"](s["a"], s["b"], s["x0"], s["out"], s["B"], s["D"], s["n"], s["layout"], s["flags"],
              torch.cuda.current_stream())
    return s["out"]


def work(case):
    """a, b and x0 read once, out written once; a multiplication and an addition per step."""
    elements = case["B"] * case["n"] * case["D"]
    x0 = 1 if case["mode"] == "positive" else case["B"] * case["D"]
    per = 2 * (2 if case["bf16"] else 4) + (8 if case["mode"] == "complex" else 4)
    return {"bytes": per * elements + 4 * x0, "flops": 2 * elements}


def tolerance(case):
    # About four times the largest error against float64 that the calls show over these ranges.  A complex
    # logarithm moves by pi where a value cancels to rounding error and comes out with the other sign: a few
    # values in ten thousand rows, more in proportion the shorter the rows are.
    if case["mode"] == "complex":
        return {"rel": 5e-4}
    if case["data"] == "slow":
        return {"rel": 1e-5}
    return {"rel": 5e-7}


def exact(case, seed):
    """x_t = a_t x_{t-1} + b_t in float64.  Time is cut into blocks that advance side by side from zero, each
    keeping its running product; then the blocks' start values are chained and added in."""
    a, b, x0 = _inputs(case, seed)
    B, n, D = case["B"], case["n"], case["D"]
    logs = case["mode"] == "logs"
    length = min(n, 8192)
    blocks = -(-n // length)
    bnd = case["layout"] == "BND"

    def by_step(v, fill):  # -> [length, blocks, B * D], time padded with `fill`
        v = v.double()
        if logs:
            v = v.exp_()
        v = v if bnd else v.transpose(1, 2)
        if blocks * length > n:
            v = torch.cat([v, torch.full((B, blocks * length - n, D), fill, dtype=v.dtype, device=v.device)], 1)
        return v.reshape(B, blocks, length, D).permute(2, 1, 0, 3).reshape(length, blocks, B * D).contiguous()

    product, value = by_step(a, 1.0), by_step(b, 0.0)
    del a, b
    for t in range(1, length):
        value[t].addcmul_(product[t], value[t - 1])
        product[t].mul_(product[t - 1])
    start = x0.double()
    if logs:
        start = start.exp()
    start = start.expand(B * D)
    starts = []
    for k in range(blocks):
        starts.append(start)
        start = product[-1, k] * start + value[-1, k]
    value.addcmul_(product, torch.stack(starts).unsqueeze(0))
    del product
    x = value.reshape(length, blocks, B, D).permute(2, 1, 0, 3).reshape(B, blocks * length, D)[:, :n]
    if not bnd:
        x = x.transpose(1, 2)
    if logs:
        x = x.log()
    elif case["mode"] == "complex":
        x = torch.stack([x.abs().log(), torch.where(x < 0, math.pi, 0.0).to(x.dtype)], -1)
    return x.contiguous()
