"""What this library is timed on: the linear layers of a decoder (rotate + quantize, then the FP4 product), the conversion of
tensors to FP4 and back, and the offline MR-GPTQ steps, each through the public Python binding as the README shows it.

A case is a plain dict.  `op` says what a pass does:

  linear   every linear of a decoder layer: fp4_rotate_quantize (or, `rotation` "dct", fp4_rotate_quantize_dense), fp4_gemm
  fused    the same in one call per linear, for a handful of tokens: fp4_fused_linear (MXFP4)
  w4a16    the weight-only form of that: fp4_w4a16_linear (MXFP4)
  convert  a tensor quantized to canonical codes and scales and decoded to bf16 again: what an emulated evaluation does
  hessian  fp4_gptq_accumulate_hessian of a batch of calibration rows
  gptq     fp4_gptq_prepare of a layer's Hessian, then fp4_gptq_quantize_weights

The decoder layer has `hidden` features, a q/k/v projection of `qkv` columns, a square output projection, a gate and up
projection of 2 x `inter` columns and a down projection from `inter`; with `part` "proj" it is the square projection alone.
"""
import math

import torch

from paper_2509_23202_amd import binding as fp4

FMT = {"mxfp4": fp4.MXFP4, "nvfp4": fp4.NVFP4}
GROUP = {"mxfp4": 32, "nvfp4": 16}
POLICY = {"absmax": 0, "mse": fp4.SCALE_MSE, "round43": fp4.SCALE_ROUND43, "fit": fp4.SCALE_MSE | fp4.SCALE_FIT_TENSOR}


def _layer(name, op, fmt, tokens, hidden, qkv, inter, block, part="layer", rotation="hadamard"):
    case = {"op": op, "fmt": fmt, "tokens": tokens, "hidden": hidden, "qkv": qkv, "inter": inter, "block": block,
            "part": part, "rotation": rotation}
    return dict(case, name=name) if name else case


def listed():
    return [
        # One token against one projection of the 8B-shaped layer: the smallest call, launch and host time.
        _layer("mx_proj_m1", "fused", "mxfp4", 1, 4096, 6144, 14336, 32, part="proj"),
        # Four sequences decoded with 16-bit activations, the variant for memory-bound layers.
        _layer("mx_w4a16_m4", "w4a16", "mxfp4", 4, 4096, 6144, 14336, 32),
        # Sixteen sequences decoded together: weights streamed from HBM.
        _layer("mx_decode_m16", "linear", "mxfp4", 16, 4096, 6144, 14336, 32),
        # A larger decoding batch, or a short prompt: an odd number of tokens, the wide Hadamard block.
        _layer("mx_batch_m201", "linear", "mxfp4", 201, 4096, 6144, 14336, 128),
        # A chunk of a prompt with a caller's own rotation (DCT blocks of 64), a ragged last row of tiles.
        _layer("mx_chunk_m1111_dct", "linear", "mxfp4", 1111, 4096, 6144, 14336, 64, rotation="dct"),
        # The 8B-shaped prefill, the largest ordinary MXFP4 product.
        _layer("mx_prefill_m4096", "linear", "mxfp4", 4096, 4096, 6144, 14336, 32),
        # NVFP4 on the 70B-shaped layer: decoding, a mixed batch, a prompt.
        _layer("nv_decode_m16", "linear", "nvfp4", 16, 8192, 10240, 28672, 16),
        _layer("nv_batch_m320", "linear", "nvfp4", 320, 8192, 10240, 28672, 16),
        _layer("nv_prefill_m2048", "linear", "nvfp4", 2048, 8192, 10240, 28672, 16),
        # A tensor to MXFP4 and back, as an evaluation in emulation does for every activation; an odd number of rows.
        {"name": "mx_convert_16383", "op": "convert", "fmt": "mxfp4", "rows": 16383, "cols": 8192, "block": 32, "policy": "absmax"},
        # Offline, per layer of a model: the Hessian of a batch of calibration rows, then the error-feedback quantization,
        # here onto the NVFP4 grid whose group and tensor scales were both fitted.
        {"name": "hessian_k4096", "op": "hessian", "rows": 8192, "cols": 4096, "block": 128},
        {"name": "nv_gptq_k4096", "op": "gptq", "fmt": "nvfp4", "rows": 6144, "cols": 4096, "block": 16, "policy": "fit", "act_order": True},
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    op = rng.choice(["linear", "linear", "linear", "linear", "fused", "w4a16", "convert", "hessian", "gptq"])
    fmt = rng.choice(["mxfp4", "nvfp4"])
    block = rng.choice([16, 32, 64, 128])
    if op in ("linear", "fused", "w4a16"):
        if op != "linear":
            fmt = "mxfp4"
        hidden = 128 * _log_int(rng, 8, 64)
        qkv = hidden + 8 * rng.randint(hidden // 64, hidden // 16)   # (grouped keys and values: not always whole tiles)
        inter = 128 * int(hidden / 128 * rng.uniform(2.0, 3.5))
        part = "proj" if rng.random() < 0.2 else "layer"
        case = _layer("", op, fmt, 1, hidden, qkv, inter, block, part, rng.choice(["hadamard", "hadamard", "hadamard", "dct"]) if op == "linear" else "hadamard")
        most = {"fused": 4, "w4a16": 16, "linear": 4096}[op]
        params = sum(n * k for n, k in _linears(case))
        case["tokens"] = min(_log_int(rng, 1, most), max(1, int(2048 * 8.5e8 / params)))
        return case
    if op == "convert":
        return {"op": op, "fmt": fmt, "rows": _log_int(rng, 1, 16384), "cols": 128 * _log_int(rng, 8, 64), "block": block,
                "policy": rng.choice(["absmax", "mse"] + (["round43"] if fmt == "mxfp4" else ["fit"]))}
    cols = 128 * _log_int(rng, 8, 32)
    if op == "hessian":
        return {"op": op, "rows": _log_int(rng, 256, 8192), "cols": cols, "block": block}
    return {"op": op, "fmt": fmt, "rows": 8 * _log_int(rng, 64, 768), "cols": cols, "block": block,
            "policy": rng.choice(["absmax", "mse"] + (["round43"] if fmt == "mxfp4" else ["fit"])), "act_order": rng.random() < 0.8}


def _linears(case):
    """(N, K) of the linears that a pass goes through."""
    h, i = case["hidden"], case["inter"]
    return [(h, h)] if case["part"] == "proj" else [(case["qkv"], h), (h, h), (2 * i, h), (h, i)]


def _normal(g, rows, cols):
    return torch.randn(rows, cols, device="cuda", dtype=torch.float32, generator=g)


def _activations(g, fmt, rows, cols):
    """bf16 activations: normal with 0.5 % of the channels 50 times as large, or for NVFP4 Student-t with three degrees of
    freedom scaled to unit variance."""
    x = _normal(g, rows, cols)
    if fmt == "nvfp4":
        chi2 = sum(_normal(g, rows, cols).square_() for _ in range(3))
        x /= chi2.sqrt_()   # N / sqrt(chi2 / 3), over sqrt(3)
    else:
        loud = torch.randperm(cols, device="cuda", generator=g)[: max(1, round(0.005 * cols))]
        x[:, loud] *= 50.0
    return x.to(torch.bfloat16)


def _weights(g, rows, cols, sigma=0.02):
    return torch.randn(rows, cols, device="cuda", dtype=torch.bfloat16, generator=g).mul_(sigma)


def _hadamard(b):
    h = torch.ones(1, 1, device="cuda", dtype=torch.float32)
    while h.shape[0] < b:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    return h / math.sqrt(b)


def _dct(b):
    n = torch.arange(b, device="cuda", dtype=torch.float32)
    m = torch.cos(math.pi / b * (n[:, None] + 0.5) * n[None, :]) * math.sqrt(2.0 / b)
    m[:, 0] = math.sqrt(1.0 / b)
    return m.to(torch.bfloat16).contiguous()


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    op = case["op"]
    if op in ("linear", "fused", "w4a16"):
        fmt = FMT[case["fmt"]]
        rot = _dct(case["block"]) if case["rotation"] == "dct" else None
        layer = []
        for n, k in _linears(case):
            w = _weights(g, n, k, 0.015 if case["fmt"] == "nvfp4" else 0.02)
            if rot is None:
                q = fp4.fp4_quantize_weights(w, case["block"], fmt, flags=fp4.LAYOUT_GEMM)
            else:
                q = fp4.fp4_rotate_quantize_dense(w, rot, fmt, flags=fp4.LAYOUT_GEMM)
            layer.append((_activations(g, case["fmt"], case["tokens"], k), q, n, k))
            del w
        return {"op": op, "fmt": fmt, "block": case["block"], "rot": rot, "layer": layer, "tokens": case["tokens"]}
    if op == "convert":
        return {"op": op, "fmt": FMT[case["fmt"]], "block": case["block"], "policy": POLICY[case["policy"]],
                "decode": POLICY[case["policy"]] & fp4.SCALE_ROUND43,
                "x": _activations(g, case["fmt"], case["rows"], case["cols"])}
    if op == "hessian":
        return {"op": op, "block": case["block"], "x": _activations(g, "mxfp4", case["rows"], case["cols"])}
    # A layer's Hessian X'^T X' of rotated calibration rows, half as many again as features, and its weights.
    k, b = case["cols"], case["block"]
    x = _activations(g, "mxfp4", k + k // 2, k).float()
    x = (x.view(-1, b) @ _hadamard(b)).view(-1, k)
    hessian = x.t().contiguous() @ x
    return {"op": op, "fmt": FMT[case["fmt"]], "block": b, "policy": POLICY[case["policy"]], "act_order": case["act_order"],
            "hessian": ((hessian + hessian.t()) * 0.5).contiguous(), "w": _weights(g, case["rows"], k)}


def run(state):
    op = state["op"]
    if op == "linear":
        out = []
        for x, (wc, ws, wt), n, k in state["layer"]:
            if state["rot"] is None:
                ac, asc, at = fp4.fp4_rotate_quantize(x, state["block"], state["fmt"], flags=fp4.LAYOUT_GEMM)
            else:
                ac, asc, at = fp4.fp4_rotate_quantize_dense(x, state["rot"], state["fmt"], flags=fp4.LAYOUT_GEMM)
            out.append(fp4.fp4_gemm(ac, asc, at, wc, ws, wt, state["tokens"], n, k, state["fmt"],
                                    flags=fp4.A_LAYOUT_GEMM | fp4.W_LAYOUT_GEMM))
        return out
    if op == "fused":
        return [fp4.fp4_fused_linear(x, state["block"], wc, ws, n) for x, (wc, ws, _), n, _ in state["layer"]]
    if op == "w4a16":
        return [fp4.fp4_w4a16_linear(x, state["block"], wc, ws, n) for x, (wc, ws, _), n, _ in state["layer"]]
    if op == "convert":
        x = state["x"]
        codes, scales, tensor_scale = fp4.fp4_rotate_quantize(x, state["block"], state["fmt"], flags=state["policy"])
        y = fp4.fp4_dequantize(codes, scales, tensor_scale, x.shape[0], x.shape[1], state["fmt"], flags=state["decode"])
        return {"codes": codes, "scales": scales, "tensor_scale": tensor_scale, "values": y}
    if op == "hessian":
        return fp4.fp4_gptq_accumulate_hessian(state["x"], state["block"])
    perm, factor = fp4.fp4_gptq_prepare(state["hessian"], 1e-2, state["act_order"])
    codes, scales, tensor_scale = fp4.fp4_gptq_quantize_weights(state["w"], state["block"], state["fmt"], factor, perm, flags=state["policy"])
    return {"perm": perm, "factor": factor, "codes": codes, "scales": scales, "tensor_scale": tensor_scale}


def work(case):
    op = case["op"]
    if op in ("linear", "fused", "w4a16"):
        m, per = case["tokens"], 0.5 + 1.0 / GROUP[case["fmt"]]
        pairs = _linears(case)
        return {"bytes": sum(2 * m * k + per * n * k + 2 * m * n for n, k in pairs), "flops": sum(2.0 * m * n * k for n, k in pairs)}
    t, k = case["rows"], case["cols"]
    if op == "convert":   # the input read, codes and scales written and read, the decoded tensor written
        return {"bytes": t * k * (2 + 2 * (0.5 + 1.0 / GROUP[case["fmt"]]) + 2), "flops": 2.0 * t * k * min(case["block"], 32)}
    if op == "hessian":   # one triangle of a symmetric matrix
        return {"bytes": 2.0 * t * k + 4.0 * k * k, "flops": 1.0 * t * k * (k + 1)}
    # Cholesky factor, its triangular inverse, and the push of every column's error onto the columns behind it
    return {"bytes": 8.0 * k * k + t * k * (2 + 0.5 + 1.0 / GROUP[case["fmt"]]), "flops": 2.0 * k ** 3 / 3 + 1.0 * t * k * k}


def tolerance(case):
    """About four times what the path differed by from itself with exact inputs or in 64 bits."""
    op = case["op"]
    if op in ("linear", "fused", "w4a16"):   # bf16 results against the fp64 product of the same operands: 1.7e-3, largest 3.9e-3
        return {"rel": 7e-3, "max": 2e-2}
    if op == "convert":   # 64-bit rotation, rounded once: no code differed; a searched scale may tie
        return {"rel": 1e-3, "differ": 2e-4}
    if op == "hessian":   # 64 bits: 1.4e-6, largest 6.9e-6
        return {"rel": 5e-6, "max": 3e-5}
    # factor against 64 bits: 3.5e-5, largest 2.2e-3; codes swept with the 64-bit factor: 2.4e-3 of the bytes (two codes each)
    return {"rel": 1.4e-4, "max": 9e-3, "differ": 9.6e-3}
