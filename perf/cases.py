"""The work a user of this framework has it do, as measurable cases.

A program that serves a model quantized with AMS-Quant keeps the packed weights, their scales and the
activation buffers on the GPU and calls the Linear once per layer and token, eagerly or as a captured
HIP graph; for prompts longer than AMS_MAX_M it restores a matrix to fp16 and multiplies with the
library GEMM; offline it quantizes and packs fp16 weights on the host.  The cases are these three paths:

  step     the Linears of one decode step captured as a HIP graph, replayed (one pass = one replay)
  linear   one eager call of ams_linear, ams_linear_ws, ams_linear_static_ws or ams_linear_grouped
  dequant  ams_dequant / ams_dequant_grouped of a whole matrix (prefill)
  pack     ams_pack on host memory (quantize a layer; offline)

Packed weights are made from seeded codes (absmax-scaled Gaussian rows rounded to the format, as the
quantizer would leave them, the members of a sharing group given a common last bit) by ams_pack_codes;
activations are N(0, 1).  Every Linear of a step has inputs and outputs of its own.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_16045_amd as ams

# name -> (format number, mantissa bits of a code, weights that share a last bit, record size, bits per weight)
FORMATS = {
    "fp5.33": (ams.FP533, 3, 3, 96, 16 / 3),
    "fp4.25": (ams.FP425, 2, 4, 128, 4.25),
    "fp4.5": (ams.FP45, 2, 2, 128, 4.5),
    "fp4.33": (ams.FP433, 2, 3, 96, 13 / 3),
    "fp6": (ams.FP6, 3, 1, 96, 6.0),
    "fp5": (ams.FP5, 2, 1, 128, 5.0),
    "fp4": (ams.FP4, 1, 1, 128, 4.0),
}
FMAX = {1: 6.0, 2: 7.0, 3: 7.5}  # largest magnitude by mantissa bits
MAX_WEIGHTS = 1 << 27  # of a drawn case: a quarter of the largest listed one


def listed():
    llama8b = "6144x4096,4096x4096,28672x4096,4096x14336"  # qkv, o, gate/up, down of Llama-3-8B
    return [
        # the smallest Linear of the configurations: latency of a single eager call
        {"name": "smallest_call", "op": "linear", "entry": "plain", "fmt": "fp4.25", "M": 1, "shapes": "256x768", "scale_group": 0},
        # a decoder layer of an 8B model, one sequence: the headline use
        {"name": "decode_8b_m1", "op": "step", "entry": "plain", "fmt": "fp5.33", "M": 1, "shapes": llama8b, "scale_group": 0},
        # the same with four sequences in the smaller format
        {"name": "decode_8b_m4", "op": "step", "entry": "plain", "fmt": "fp4.25", "M": 4, "shapes": llama8b, "scale_group": 0},
        # the largest batch of a decoder layer
        {"name": "decode_8b_m32", "op": "step", "entry": "plain", "fmt": "fp4.25", "M": 32, "shapes": llama8b, "scale_group": 0},
        # attention output and MLP down projections of a 70B model, eight sequences
        {"name": "decode_70b_m8", "op": "step", "entry": "plain", "fmt": "fp5.33", "M": 8, "shapes": "8192x8192,8192x28672", "scale_group": 0},
        # two MLP-down shapes of the format comparison (Qwen2.5-7B, Qwen3-4B) in a plain mini-float
        {"name": "decode_down_fp6_m1", "op": "step", "entry": "plain", "fmt": "fp6", "M": 1, "shapes": "3584x18944,2560x9728", "scale_group": 0},
        # the Qwen3-32B MLP-down at batch 16 through the entry point that splits K without allocating
        {"name": "qwen32b_down_m16", "op": "linear", "entry": "static", "fmt": "fp5.33", "M": 16, "shapes": "5120x25600", "scale_group": 0},
        # the vocabulary projection of Llama-3-8B: the largest single Linear
        {"name": "lm_head_m8", "op": "linear", "entry": "plain", "fmt": "fp4.25", "M": 8, "shapes": "128256x4096", "scale_group": 0},
        # one scale per 128 input channels
        {"name": "grouped_gate_up_m4", "op": "linear", "entry": "grouped", "fmt": "fp4.25", "M": 4, "shapes": "28672x4096", "scale_group": 128},
        # sizes that divide by nothing: rows of X that are not 16-byte aligned, ragged strips and records
        {"name": "ragged_m5", "op": "linear", "entry": "plain", "fmt": "fp5.33", "M": 5, "shapes": "11003x4099", "scale_group": 0},
        # restoration of a gate/up matrix for a long prompt's GEMM
        {"name": "dequant_gate_up", "op": "dequant", "entry": "plain", "fmt": "fp4.25", "M": 0, "shapes": "28672x4096", "scale_group": 0},
        # offline quantization of a q/o projection
        {"name": "pack_o", "op": "pack", "entry": "plain", "fmt": "fp5.33", "M": 0, "shapes": "4096x4096", "scale_group": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    n = _log_int(rng, lo, hi)
    step = rng.choice((1, 8, 64, 64, 128))  # model sizes are round numbers; one in five is not
    return max(lo, n // step * step)


def _shape(rng, max_n, most):
    while True:
        n, k = _size(rng, 256, max_n), _size(rng, 256, 28672)
        if n * k <= most:
            return n, k


def draw(rng):
    fmt = rng.choice(("fp5.33", "fp4.25", "fp5.33", "fp4.25", rng.choice(tuple(FORMATS))))
    op = rng.choice(("step", "step", "step", "linear", "linear", "linear", "dequant", "pack"))
    entry, m, scale_group = "plain", 0, 0
    if op in ("step", "linear"):
        m = _log_int(rng, 1, 32)
        entry = rng.choice(("plain", "plain", "ws", "static") if op == "step" else ("plain", "ws", "static", "grouped"))
    elif op == "dequant":
        entry = rng.choice(("plain", "grouped"))
    if entry == "grouped":
        scale_group = FORMATS[fmt][3] << rng.randrange(0, 3)
    if op == "step":  # a decoder layer: qkv, o, gate/up, down of some model
        hidden = _size(rng, 768, 8192)
        kv = max(64, hidden // rng.choice((1, 4, 8)))
        ffn = int(hidden * rng.uniform(2.5, 4.0)) // 64 * 64
        shapes = [(hidden + 2 * kv, hidden), (hidden, hidden), (2 * ffn, hidden), (hidden, ffn)]
        while sum(n * k for n, k in shapes) > MAX_WEIGHTS:
            shapes.remove(max(shapes, key=lambda s: s[0] * s[1]))
    elif op == "pack":
        shapes = [_shape(rng, 28672, 1 << 24)]
    else:
        shapes = [_shape(rng, 8192 if entry == "static" else 131072, MAX_WEIGHTS)]
    return {"op": op, "entry": entry, "fmt": fmt, "M": m, "shapes": ",".join("%dx%d" % s for s in shapes), "scale_group": scale_group}


def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split(",")]


def _generator(seed, i):
    return torch.Generator(device="cuda").manual_seed((seed * 1009 + i) % (1 << 62))


def _row_chunks(n, k, most=1 << 25):
    step = max(16, most // k // 16 * 16)
    return [(r, min(n, r + step)) for r in range(0, n, step)]


def _magnitude(code, mbits):
    e, m = code >> mbits, code & ((1 << mbits) - 1)
    return torch.where(e == 0, m.double(), (m + (1 << mbits)).double() * torch.exp2((e - 1).double())) * 2.0**-mbits


def _quantized(case, i, seed):
    """Codes [N, K] (uint8) of Linear i and its fp16 scales: [N], or [N, runs] with one per run of input channels."""
    _, mbits, group, _, _ = FORMATS[case["fmt"]]
    n, k = _shapes(case)[i]
    gen = _generator(seed, 2 * i)
    runs = -(-k // case["scale_group"]) if case["scale_group"] else 1
    width = case["scale_group"] or k
    codes = torch.empty((n, k), dtype=torch.uint8, device="cuda")
    scales = torch.empty((n, runs), dtype=torch.float16, device="cuda")
    one = 1 << mbits
    for r0, r1 in _row_chunks(n, k):
        w = torch.randn((r1 - r0, runs * width), generator=gen, device="cuda") * 0.02
        w = w.view(r1 - r0, runs, width)
        s = (w.abs().amax(2) / FMAX[mbits]).to(torch.float16)
        scales[r0:r1] = s
        t = (w.abs() / s.float().unsqueeze(2)).view(r1 - r0, -1)[:, :k]
        code = torch.where(
            t < 2, torch.round(t * one), torch.where(t < 4, one + torch.round(t * (one / 2)), 2 * one + torch.round(t * (one / 4)))
        )
        code = code.clamp_(max=4 * one - 1).to(torch.uint8)
        if group > 1:  # the members of a group take the first one's last bit
            first = torch.arange(k, device="cuda") // group * group
            code = (code & 0xFE) | (code[:, first] & 1)
        codes[r0:r1] = code | ((w.view(r1 - r0, -1)[:, :k] < 0).to(torch.uint8) << (mbits + 2))
    return codes, scales if case["scale_group"] else scales.view(n)


def _activations(case, i, seed):
    _, k = _shapes(case)[i]
    return torch.randn((case["M"], k), generator=_generator(seed, 2 * i + 1), device="cuda").to(torch.float16)


def _host_weights(case, seed):
    (n, k), = _shapes(case)
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((n, k), dtype=np.float32) * np.float32(0.02)).astype(np.float16)


def _call(case, p):
    fmt, n = p["fmt"], p["N"]
    if case["entry"] == "ws":
        return ams.ams_linear_ws(p["W"], p["scales"], p["X"], n, fmt, p["workspace"], out=p["Y"])
    if case["entry"] == "static":
        return ams.ams_linear_static_ws(p["W"], p["scales"], p["X"], n, fmt, out=p["Y"])
    if case["entry"] == "grouped":
        return ams.ams_linear_grouped(p["W"], p["scales"], case["scale_group"], p["X"], n, fmt, out=p["Y"])
    return ams.ams_linear(p["W"], p["scales"], p["X"], n, fmt, out=p["Y"])


def prepare(case, seed):
    if case["op"] == "pack":
        return {"case": case, "W": _host_weights(case, seed)}
    ams.ams_init()
    fmt = FORMATS[case["fmt"]][0]
    linears = []
    for i, (n, k) in enumerate(_shapes(case)):
        codes, scales = _quantized(case, i, seed)
        packed = torch.from_numpy(ams.ams_pack_codes(fmt, codes.cpu().numpy())).cuda()
        if case["scale_group"]:  # the order the kernels read: [strip of 16 rows][run][row inside the strip], 1.0 for padding rows
            strips, runs = -(-n // 16), scales.shape[1]
            padded = torch.ones((strips * 16, runs), dtype=torch.float16, device="cuda")
            padded[:n] = scales
            scales = padded.view(strips, 16, runs).transpose(1, 2).contiguous()
        p = {"fmt": fmt, "N": n, "K": k, "W": packed, "scales": scales}
        if case["op"] == "dequant":
            p["Y"] = torch.empty((n, k), dtype=torch.float16, device="cuda")
        else:
            p["X"] = _activations(case, i, seed)
            p["Y"] = torch.empty((case["M"], n), dtype=torch.float16, device="cuda")
        linears.append(p)
    if case["entry"] == "ws":  # one workspace for the Linears of a step: they run one after the other
        need = max(ams.ams_linear_workspace_bytes(fmt, case["M"], p["N"], p["K"]) for p in linears)
        workspace = torch.zeros(max(need, 16), dtype=torch.uint8, device="cuda")
        for p in linears:
            p["workspace"] = workspace
    state = {"case": case, "linears": linears}
    if case["op"] == "step":
        for p in linears:
            _call(case, p)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            for p in linears:
                _call(case, p)
    return state


def run(state):
    case = state["case"]
    if case["op"] == "pack":
        return list(ams.ams_pack(FORMATS[case["fmt"]][0], state["W"]))
    if case["op"] == "step":
        state["graph"].replay()
        return [p["Y"] for p in state["linears"]]
    (p,) = state["linears"]
    if case["op"] == "dequant":
        if case["entry"] == "grouped":
            return ams.ams_dequant_grouped(p["fmt"], p["W"], p["scales"], case["scale_group"], p["N"], p["K"], out=p["Y"])
        return ams.ams_dequant(p["fmt"], p["W"], p["scales"], p["N"], p["K"], out=p["Y"])
    return _call(case, p)


def work(case):
    bits = FORMATS[case["fmt"]][4]
    total, flops = 0.0, 0.0
    for n, k in _shapes(case):
        runs = -(-k // case["scale_group"]) if case["scale_group"] else 1
        total += n * k * bits / 8 + 2 * n * runs  # packed weights and scales
        if case["op"] in ("dequant", "pack"):
            total += 2 * n * k
        else:
            total += 2 * case["M"] * (n + k)
            flops += 2.0 * case["M"] * n * k
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["op"] in ("dequant", "pack"):
        return "exact"  # one rounding of an exact product; whole bytes
    # fp32 sums rounded to fp16 once: 2.1e-4 from the 64-bit result; two orders of the sums differ in the last bit of some results
    return {"rel": 8e-4, "max": 4e-3}


def exact(case, seed):
    if case["op"] == "pack":
        w = np.abs(_host_weights(case, seed).astype(np.float64))
        return [None, w.max(1) / FMAX[FORMATS[case["fmt"]][1]]]
    mbits = FORMATS[case["fmt"]][1]
    outs = []
    for i, (n, k) in enumerate(_shapes(case)):
        codes, scales = _quantized(case, i, seed)
        x = _activations(case, i, seed).double() if case["op"] != "dequant" else None
        out = torch.empty((n, k) if x is None else (case["M"], n), dtype=torch.float64, device="cuda")
        for r0, r1 in _row_chunks(n, k):
            code = codes[r0:r1].int()
            v = _magnitude(code & ((4 << mbits) - 1), mbits)
            v = torch.where((code >> (mbits + 2)) > 0, -v, v)
            s = scales[r0:r1].double()
            v *= s.repeat_interleave(case["scale_group"], 1)[:, :k] if case["scale_group"] else s.unsqueeze(1)
            if x is None:
                out[r0:r1] = v
            else:
                out[:, r0:r1] = x @ v.t()
        outs.append(out)
    return outs if case["op"] == "step" else outs[0]
