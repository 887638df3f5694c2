"""What this library is used for, as cases that can be timed: forward, input gradient and weight gradient of the
depthwise convolution through the calls of ``paper_2604_25422_amd.binding``, on torch device tensors.

A case is a dict: ``B, C, L, K, pad`` and ``dtype`` ("f32" or "bf16") as the library takes them, ``calls``, which is how
a program makes its pass - "fwd" (inference), "separate" (``dwconv_fwd``, ``dwconv_bwd_input``, ``dwconv_bwd_weight``) or
"fused" (``dwconv_fwd`` and ``dwconv_bwd``, both gradients in one call) - and ``filter``, the distribution of the taps.
"""
import math

import torch

from paper_2604_25422_amd import binding

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
ELEM = {"f32": 4, "bf16": 2}


def _case(name, B, C, L, K, pad, dtype, calls, filt="normal"):
    return {"name": name, "B": B, "C": C, "L": L, "K": K, "pad": pad, "dtype": dtype, "calls": calls, "filter": filt}


def listed():
    return [
        # a training step so small that launches and the way to them are what it costs (the small configuration)
        _case("small_f32", 4, 64, 1024, 16, 15, "f32", "separate"),
        # inference on one sequence at the headline's width and length
        _case("serve_one_f32", 1, 256, 4096, 64, 63, "f32", "fwd"),
        # the headline training step, its three paths one by one as the benchmark line reports them
        _case("headline_f32", 32, 256, 4096, 64, 63, "f32", "separate"),
        # short centred filter, as in convolutional mixers; both gradients in one call
        _case("short_filter_f32", 64, 512, 2048, 7, 3, "f32", "fused"),
        # state-space kernels materialised over the whole sequence
        _case("long_filter_f32", 8, 256, 8192, 8192, 8191, "f32", "separate", "decay"),
        _case("long_filter_bf16", 8, 256, 8192, 8192, 8191, "bf16", "separate", "decay"),
        # mixed-precision training at a transformer's width
        _case("train_bf16", 128, 768, 1024, 32, 31, "bf16", "fused"),
        # the shape of the paper's measurements: two million rows of 48 hours, pad K / 2, in either storage type
        _case("paper_f32", 16384, 128, 48, 48, 24, "f32", "fused"),
        _case("paper_bf16", 16384, 128, 48, 48, 24, "bf16", "fused"),
        # a filter of an eighth of a thousand taps on the headline's tensor
        _case("mid_filter_f32", 32, 256, 4096, 128, 127, "f32", "separate"),
        # many short windows with a filter as long as the window
        _case("global_filter_f32", 2048, 128, 256, 256, 255, "f32", "separate"),
        # a sequence length nobody rounded, in bf16
        _case("odd_length_bf16", 32, 256, 4097, 64, 63, "bf16", "fused"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Any of the above ranges: rows of 24 to 8192 positions (odd ones among them), filters of 3 taps to the whole row,
    a quarter of a million to a hundred million elements, either type, each way of calling."""
    dtype = rng.choice(("f32", "f32", "bf16"))
    calls = rng.choice(("fwd", "separate", "fused"))
    L = _log_int(rng, 24, 8192)
    if rng.random() < 0.5:                      # half of the lengths are multiples of 16, as programs like them
        L = max(32, L // 16 * 16)
    kind = rng.random()
    if kind < 0.6:
        K = _log_int(rng, 3, 64)
    elif kind < 0.8:
        K = _log_int(rng, 65, 256)
    else:
        K = L
    pad = rng.choice((K - 1, K // 2))
    C = _log_int(rng, 32, 768)
    if rng.random() < 0.5:
        C = max(32, C // 32 * 32)
    top = 1e8
    if K > 64:
        top = min(top, 2.0 ** 24 * 8192 / 4 / K)     # the work of a quarter of the listed long filter
    elems = math.exp(rng.uniform(math.log(2.0 ** 18), math.log(max(top, 2.0 ** 19))))
    B = max(1, int(elems / (C * L)))
    return {"B": B, "C": C, "L": L, "K": K, "pad": pad, "dtype": dtype, "calls": calls,
            "filter": "decay" if K > 256 else "normal"}


def _inputs(case, seed):
    """x, dy ~ N(0, 1); taps ~ N(0, 1 / K), or of long filters exp(-a k) cos(b k) as a state-space model's kernel."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, C, L, K, dt = case["B"], case["C"], case["L"], case["K"], DTYPES[case["dtype"]]

    def normal(*shape):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)

    x = normal(B, C, L).to(dt)
    dy = normal(B, C, L).to(dt) if case["calls"] != "fwd" else None
    if case["filter"] == "decay":
        a = 1e-4 + (1e-2 - 1e-4) * torch.rand(C, 1, generator=g, device="cuda", dtype=torch.float64)
        b = math.pi * torch.rand(C, 1, generator=g, device="cuda", dtype=torch.float64)
        k = torch.arange(K, device="cuda", dtype=torch.float64)
        w = (torch.exp(-a * k) * torch.cos(b * k)).to(dt)
    else:
        w = (normal(C, K) / math.sqrt(K)).to(dt)
    return x, w, dy


def prepare(case, seed):
    """Inputs, and the weight-gradient workspace that a training program keeps next to its layer."""
    x, w, dy = _inputs(case, seed)
    ws = binding.new_workspace(x, case["K"], case["pad"]) if case["calls"] != "fwd" else None
    return {"x": x, "w": w, "dy": dy, "ws": ws, "K": case["K"], "pad": case["pad"], "calls": case["calls"]}


def run(state):
    x, w, dy, ws, pad = state["x"], state["w"], state["dy"], state["ws"], state["pad"]
    out = {"y": binding.dwconv_fwd(x, w, pad)}
    if state["calls"] == "separate":
        out["dx"] = binding.dwconv_bwd_input(dy, w, pad)
        out["dw"] = binding.dwconv_bwd_weight(x, dy, state["K"], pad, workspace=ws)
    elif state["calls"] == "fused":
        out["dx"], out["dw"] = binding.dwconv_bwd(dy, x, w, pad, workspace=ws)
    return out


def work(case):
    """Per call: every tensor it takes read once, every tensor it returns written once; two operations for each product
    of a tap and a position inside the row, in every path."""
    B, C, L, K, pad = case["B"], case["C"], case["L"], case["K"], case["pad"]
    n, ck = B * C * L, C * K
    tensors, filters, paths = {"fwd": (2, 1, 1), "separate": (6, 3, 3), "fused": (5, 3, 3)}[case["calls"]]
    pairs = sum(max(0, L - abs(j - pad)) for j in range(K))
    return {"bytes": ELEM[case["dtype"]] * (tensors * n + filters * ck), "flops": paths * 2 * B * C * pairs}


def tolerance(case):
    """fp32: products and sums in 32 bits, in any order.  bf16: 32-bit sums of exact products, one rounding at the end."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    return {"rel": 4e-3, "max": 1.6e-2}


def exact(case, seed):
    x, w, dy = _inputs(case, seed)
    L, K, pad = case["L"], case["K"], case["pad"]
    x, w = x.double(), w.double()
    y = torch.zeros_like(x)
    if dy is not None:
        dy = dy.double()
        dx, dw = torch.zeros_like(x), torch.zeros_like(w)
    for j in range(K):
        o = j - pad                              # y[t] takes x[t + o]
        a, b = max(0, -o), min(L, L - o)
        if a >= b:
            continue
        wj = w[:, j:j + 1]
        y[..., a:b].addcmul_(x[..., a + o:b + o], wj)
        if dy is not None:
            dx[..., a + o:b + o].addcmul_(dy[..., a:b], wj)
            dw[:, j] = (dy[..., a:b] * x[..., a + o:b + o]).sum(dim=(0, 2))
    return {"y": y} if dy is None else {"y": y, "dx": dx, "dw": dw}
