"""Performance cases of the Huffman weight codec and its fused decode-GEMV.

A case is a dict of plain values; `op` names the entry points it goes through:

  gemv    DeviceTensor.gemv: one matrix times 1 to 16 activation rows
  mlp     gemv_multi (gate and up, one launch) and gemv (down)
  layer   gemv_multi (q, k, v), gemv (o), gemv_multi (gate, up), gemv (down):
          one decode step through every matrix of a decoder layer
  gemm    DeviceTensor.gemm: a prefill of many activation rows
  decode  DeviceTensor.decode: the whole matrix back to 16-bit weights
  encode  encode: codebook and container of a host matrix

`format` is the container format: "split" (bf16, the default of encode),
"whole" (bf16, whole-exponent code) or "fp16". The listed sizes are those of
this repository's workloads (gen/synth.py), with ragged ones of its tests;
draw() covers rows of 256 to 28672 and columns of 512 to 28672 (multiples of 8,
which the container asks for), 1 to 16 activation rows in a decode step and 1
to 512 in a prefill, in every format.
"""
from __future__ import annotations

import numpy as np
import torch

import paper_2502_00922_amd as hl

ENCODE = {"split": {}, "whole": {"whole_exponent": True}, "fp16": {"fp16": True}}
# container bits per weight on these weights (64-weight segments)
CONTAINER_BITS = {"split": 11.77, "whole": 10.84, "fp16": 11.09}
X_TYPE = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}
MOST_WEIGHTS = 128 << 20  # of a drawn case


def listed():
    return [
        # the smallest product, float32 activations: launch and latency
        {"name": "gemv 1024x1024 f32", "op": "gemv", "format": "split", "rows": 1024, "cols": 1024, "batch": 1,
         "x": "f32"},
        # one attention projection of a 7B or 8B model, one token
        {"name": "gemv 4096x4096", "op": "gemv", "format": "split", "rows": 4096, "cols": 4096, "batch": 1,
         "x": "bf16"},
        # a narrow projection with a ragged last row block, a few tokens at once
        {"name": "gemv 1000x4096 b3", "op": "gemv", "format": "split", "rows": 1000, "cols": 4096, "batch": 3,
         "x": "bf16"},
        # a float16 release of a model: its widest matrix, one token
        {"name": "gemv fp16 14336x4096", "op": "gemv", "format": "fp16", "rows": 14336, "cols": 4096, "batch": 1,
         "x": "f16"},
        # the MLP of a 7B model (odd multiple of the tile: 688 row blocks, 172 segments), a full batch, in the
        # smaller container
        {"name": "mlp 7b whole b16", "op": "mlp", "format": "whole", "hidden": 4096, "inter": 11008, "batch": 16},
        # a decode step through one layer of an 8B model, a batch of 8
        {"name": "layer 8b b8", "op": "layer", "format": "split", "hidden": 4096, "kv": 1024, "inter": 14336,
         "batch": 8},
        # a decode step through one layer of a 70B model, one token: the headline workload's layer
        {"name": "layer 70b b1", "op": "layer", "format": "split", "hidden": 8192, "kv": 1024, "inter": 28672,
         "batch": 1},
        # a short prompt
        {"name": "prefill 4096x14336 t48", "op": "gemm", "format": "split", "rows": 4096, "cols": 14336,
         "tokens": 48},
        # a longer prompt
        {"name": "prefill 14336x4096 t512", "op": "gemm", "format": "split", "rows": 14336, "cols": 4096,
         "tokens": 512},
        # a matrix expanded for a consumer that wants plain weights
        {"name": "decode 28672x8192", "op": "decode", "format": "split", "rows": 28672, "cols": 8192},
        {"name": "decode fp16 4096x11008", "op": "decode", "format": "fp16", "rows": 4096, "cols": 11008},
        # the offline step: compressing one matrix on the host
        {"name": "encode 4096x4096", "op": "encode", "format": "split", "rows": 4096, "cols": 4096},
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def _shape(rng, step):
    """Rows of any number and columns of a multiple of `step`."""
    cols = step * max(1, round(_spread(rng, 512, 28672) / step))
    rows = _spread(rng, 256, min(28672, MOST_WEIGHTS // cols))
    return (rows - rows % 16 if rng.random() < 0.5 and rows >= 272 else rows), cols


def draw(rng):
    op = rng.choices(["gemv", "mlp", "layer", "gemm", "decode", "encode"], [6, 2, 1, 3, 2, 1])[0]
    fmt = rng.choices(["split", "whole", "fp16"], [3, 1, 1])[0]
    if op == "gemv":
        # the float16 product and the matrix cores take 4 segments a group: multiples of 256 give those
        step = 256 if fmt == "fp16" or rng.random() < 0.6 else rng.choice([8, 64])
        rows, cols = _shape(rng, step)
        x = "f16" if fmt == "fp16" else rng.choices(["bf16", "f32"], [3, 1])[0]
        return {"op": op, "format": fmt, "rows": rows, "cols": cols, "batch": _spread(rng, 1, 16), "x": x}
    if op == "mlp":
        hidden = 256 * rng.randint(4, 20)
        return {"op": op, "format": fmt, "hidden": hidden, "inter": 256 * round(hidden * rng.uniform(2.5, 4) / 256),
                "batch": _spread(rng, 1, 16)}
    if op == "layer":
        hidden = 256 * rng.randint(4, 16)
        return {"op": op, "format": fmt, "hidden": hidden, "kv": hidden // rng.choice([1, 2, 4]),
                "inter": 256 * round(hidden * rng.uniform(2.5, 3.5) / 256), "batch": _spread(rng, 1, 16)}
    if op == "gemm":
        rows, cols = _shape(rng, 256)  # the prefill product takes the same groups
        return {"op": op, "format": "split" if fmt == "fp16" else fmt, "rows": rows, "cols": cols,
                "tokens": _spread(rng, 1, 512)}
    rows, cols = _shape(rng, rng.choice([8, 64, 256]))
    return {"op": op, "format": fmt, "rows": rows, "cols": cols}


def _matrices(case):
    """Names, rows and columns of a case's matrices, in the order of their seeds."""
    if case["op"] not in ("mlp", "layer"):
        return [("w", case["rows"], case["cols"])]
    h, f = case["hidden"], case["inter"]
    mlp = [("gate", f, h), ("up", f, h), ("down", h, f)]
    if case["op"] == "mlp":
        return mlp
    return [("q", h, h), ("k", case["kv"], h), ("v", case["kv"], h), ("o", h, h)] + mlp


def _inputs(case):
    """Names and columns of a case's activations."""
    if case["op"] == "mlp":
        return [("mlp", case["hidden"]), ("down", case["inter"])]
    if case["op"] == "layer":
        return [("attn", case["hidden"]), ("o", case["hidden"]), ("mlp", case["hidden"]), ("down", case["inter"])]
    return [("x", case["cols"])]


def _generator(seed, k):
    return torch.Generator(device="cuda").manual_seed(seed * 64 + k)


def _weights(case, seed, k, rows, cols):
    """Weights of a trained layer's kind: a narrow Gaussian bulk whose scale varies by row, 0.1% outliers 20 times
    as large, rounded to bfloat16 (then to float16 for that format: the release of a model trained in bfloat16)."""
    g = _generator(seed, k)
    w = torch.randn((rows, cols), generator=g, device="cuda").mul_(0.02)
    w.mul_(torch.randn((rows, 1), generator=g, device="cuda").mul_(0.3).exp_())
    w[torch.rand((rows, cols), generator=g, device="cuda") < 0.001] *= 20
    w = w.to(torch.bfloat16)
    return w.to(torch.float16) if case["format"] == "fp16" else w


def _activations(case, seed, k, cols):
    rows = case["tokens"] if case["op"] == "gemm" else case["batch"]
    kind = case.get("x") or ("f16" if case["format"] == "fp16" else "bf16")
    return torch.randn((rows, cols), generator=_generator(seed, 32 + k), device="cuda").to(X_TYPE[kind])


def _bits(w):
    return w.view(torch.int16).cpu().numpy().view(np.uint16)


def prepare(case, seed):
    state = {"op": case["op"], "format": case["format"]}
    if case["op"] == "encode":
        state["w"] = _bits(_weights(case, seed, 0, case["rows"], case["cols"]))
        state["shard"] = np.zeros(state["w"].nbytes + (64 << 10), dtype=np.uint8)  # where a checkpoint is put together
        return state
    for k, (name, rows, cols) in enumerate(_matrices(case)):
        blob = hl.encode(_bits(_weights(case, seed, k, rows, cols)), **ENCODE[case["format"]])
        state[name] = hl.DeviceTensor(blob)
    if case["op"] == "decode":
        state["out"] = torch.empty((case["rows"], case["cols"]), dtype=torch.int16, device="cuda")
        return state
    state["x"] = {name: _activations(case, seed, k, cols) for k, (name, cols) in enumerate(_inputs(case))}
    # a model's program keeps the outputs of its layers
    batch = case["tokens"] if case["op"] == "gemm" else case["batch"]
    state["y"] = {name: torch.empty((batch, rows), device="cuda") for name, rows, _ in _matrices(case)}
    return state


def run(state):
    op = state["op"]
    if op == "encode":
        blob = hl.encode(state["w"], **ENCODE[state["format"]])
        state["shard"][:blob.size] = blob
        return state["shard"]
    if op == "decode":
        return state["w"].decode(state["out"])
    x, y = state["x"], state["y"]
    if op == "gemv":
        state["w"].gemv(x["x"], y["w"])
    elif op == "gemm":
        state["w"].gemm(x["x"], y["w"])
    else:
        if op == "layer":
            hl.gemv_multi([state["q"], state["k"], state["v"]], x["attn"], [y["q"], y["k"], y["v"]])
            state["o"].gemv(x["o"], y["o"])
        hl.gemv_multi([state["gate"], state["up"]], x["mlp"], [y["gate"], y["up"]])
        state["down"].gemv(x["down"], y["down"])
    return y


def work(case):
    container = CONTAINER_BITS[case["format"]] / 8
    weights = sum(rows * cols for _, rows, cols in _matrices(case))
    if case["op"] in ("decode", "encode"):
        return {"bytes": weights * (2 + container), "flops": 0}
    batch = case["tokens"] if case["op"] == "gemm" else case["batch"]
    x_bytes = 4 if case.get("x") == "f32" else 2
    ends = sum(cols for _, cols in _inputs(case)) * x_bytes + sum(rows for _, rows, _ in _matrices(case)) * 4
    return {"bytes": weights * container + batch * ends, "flops": 2 * weights * batch}


def tolerance(case):
    if case["op"] in ("decode", "encode"):
        return "exact"
    # products of 16-bit weights summed in float32: 1e-7 to 4e-7 off the sums in 64 bits, four times the largest
    return {"rel": 1.6e-6}


def exact(case, seed):
    if case["op"] == "encode":
        return None
    if case["op"] == "decode":
        return _weights(case, seed, 0, case["rows"], case["cols"]).view(torch.int16)
    inputs = {name: _activations(case, seed, k, cols).double() for k, (name, cols) in enumerate(_inputs(case))}
    source = {"w": "x", "q": "attn", "k": "attn", "v": "attn", "o": "o", "gate": "mlp", "up": "mlp", "down": "down"}
    out = {}
    for k, (name, rows, cols) in enumerate(_matrices(case)):
        w, x = _weights(case, seed, k, rows, cols), inputs[source[name]]
        out[name] = torch.cat([x @ part.double().t() for part in w.split(4096)], dim=1)
    return out
