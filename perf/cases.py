"""What this library is timed on: the calls that a program using it makes, over the range of sizes it makes them at.

The sizes of the listed cases are those of the repository's configurations (LLaMA-shaped linear layers, the
34B-class decoder block, the feed-forward shapes of the paper's kernel table) or generic (a ragged batch, a
longer prompt); `draw` spreads over the same ranges.  Weights, activations and their distributions are those of
`paper_2312_08583_amd.inputs`: fp16 N(0, sigma^2) weights with 0.1 % of entries times ten, N(0, 1) activations.

A case is one of
  linear      one layer, Y = X W^T, in one of the weight formats
  block       the seven linear layers of a decoder block at one height M: q, k, v in one grouped call, o, gate and
              up in one grouped call, down
  quantize    the offline step: fp16 weight -> planes and scales
  dequantize  planes and scales -> fp16 weight
and the formats are fp6 (row scales), fgq (one scale per `block` elements of a row), fp5 (4+1 planes), v2 (plane
layout 2) and bf16 (plane layout 2 against bf16 activations).
"""
import math

import torch

import paper_2312_08583_amd as P
from paper_2312_08583_amd import inputs

_QUANTIZE = {"fp6": P.fp6_quantize_pack, "fp5": P.fp5_quantize_pack, "v2": P.fp6_quantize_pack_v2,
             "bf16": P.fp6_quantize_pack_v2}
_DEQUANTIZE = {"fp6": P.fp6_dequantize, "fp5": P.fp5_dequantize, "v2": P.fp6_dequantize_v2, "bf16": P.fp6_dequantize_v2}
_LINEAR = {"fp6": P.fp6_linear, "fp5": P.fp5_linear, "v2": P.fp6_linear_v2, "bf16": P.fp6_linear_v2_bf16}
_WORKSPACE = {"fp6": P.fp6_linear_workspace_bytes, "fp5": P.fp5_linear_workspace_bytes,
              "v2": P.fp6_linear_v2_workspace_bytes, "bf16": P.fp6_linear_v2_workspace_bytes}
_PLANE_BYTES = {"fp6": 0.75, "fgq": 0.75, "fp5": 0.625, "v2": 0.75, "bf16": 0.75}      # per weight


def _linear_case(name, fmt, M, N, K, block=0):
    return {"name": name, "op": "linear", "fmt": fmt, "M": M, "N": N, "K": K, "block": block}


def _block_case(name, M, hidden, kv, mlp):
    return {"name": name, "op": "block", "fmt": "fp6", "M": M, "hidden": hidden, "kv": kv, "mlp": mlp}


def _offline_case(name, op, fmt, N, K, block=0):
    return {"name": name, "op": op, "fmt": fmt, "N": N, "K": K, "block": block}


def listed():
    return [
        # one small layer, one token: nothing but launch and latency
        _linear_case("lin_1024x1024_m1", "fp6", 1, 1024, 1024),
        # decoding four sequences through a 7B-shaped block
        _block_case("block_7b_m4", 4, 4096, 4096, 11008),
        # decoding one sequence through the 34B-class block (519 MB of planes: always cold)
        _block_case("block_34b_m1", 1, 8192, 1024, 22016),
        # fine-grained scales, batch 8, as in the paper's kernel table
        _linear_case("fgq128_5120x13824_m8", "fgq", 8, 5120, 13824, 128),
        # five-bit weights, batch 16
        _linear_case("fp5_28672x8192_m16", "fp5", 16, 28672, 8192),
        # a decode batch beyond one block of 16 rows
        _linear_case("lin_13824x5120_m32", "fp6", 32, 13824, 5120),
        # a ragged batch between decoding and prefill
        _linear_case("lin_8192x28672_m100", "fp6", 100, 8192, 28672),
        # a ragged prompt with bf16 activations
        _linear_case("bf16_13824x5120_m333", "bf16", 333, 13824, 5120),
        # prefill of 512 tokens
        _linear_case("lin_22016x8192_m512", "fp6", 512, 22016, 8192),
        # prefill of 2048 tokens through the 34B-class block: the largest
        _block_case("block_34b_m2048", 2048, 8192, 1024, 22016),
        # the offline step on a 70B-shaped layer
        _offline_case("quantize_28672x8192", "quantize", "fp6", 28672, 8192),
        # planes back to an fp16 weight
        _offline_case("dequantize_13824x5120", "dequantize", "fp6", 13824, 5120),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log_size(rng, lo, hi, step):
    return max(1, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step))) * step


def _log_layer(rng, step_k):
    """N and K of one layer: no more weights than 28672 x 8192."""
    N = _log_size(rng, 1024, 28672, 64)
    return N, _log_size(rng, 1024, min(28672, 28672 * 8192 // N), step_k)


def draw(rng):
    kind = rng.random()
    if kind < 0.6:
        fmt = rng.choice(["fp6", "fp6", "fp6", "fp6", "fgq", "fgq", "fp5", "fp5", "v2", "bf16", "bf16"])
        block = rng.choice([64, 128, 256]) if fmt == "fgq" else 0
        N, K = _log_layer(rng, block or 64)
        return {"op": "linear", "fmt": fmt, "M": _log_int(rng, 1, 4096), "N": N, "K": K, "block": block}
    if kind < 0.75:
        hidden = _log_size(rng, 1024, 7168, 128)
        return {"op": "block", "fmt": "fp6", "M": _log_int(rng, 1, 2048), "hidden": hidden,
                "kv": rng.choice([hidden, 1024]), "mlp": _log_size(rng, 2 * hidden, 2.7 * hidden, 64)}
    op = "quantize" if kind < 0.9 else "dequantize"
    fmt = rng.choice(["fp6", "fp6", "fgq", "fp5", "v2"])
    block = rng.choice([64, 128, 256]) if fmt == "fgq" else 0
    N, K = _log_layer(rng, block or 64)
    return {"op": op, "fmt": fmt, "N": N, "K": K, "block": block}


# ---- a user's program: weights quantized once, workspace and outputs kept

def _weight(N, K, seed):
    return inputs.weight(N, K, seed, sigma=0.02, outlier_frac=0.001, device="cuda")


def _packed(case, N, K, seed):
    W = _weight(N, K, seed)
    return P.fp6_quantize_pack_fgq(W, case["block"]) if case["fmt"] == "fgq" else _QUANTIZE[case["fmt"]](W)


def _zeros(nbytes):
    return torch.zeros(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def _block_shapes(case):
    h, kv, mlp = case["hidden"], case["kv"], case["mlp"]
    return [("q", h, h), ("k", kv, h), ("v", kv, h), ("o", h, h), ("gate", mlp, h), ("up", mlp, h), ("down", h, mlp)]


def prepare(case, seed):
    seed = inputs.BASE_SEED + 1000 * seed
    op, fmt = case["op"], case["fmt"]
    if op == "quantize":
        return {"case": case, "W": _weight(case["N"], case["K"], seed)}
    if op == "dequantize":
        return {"case": case, "planes": _packed(case, case["N"], case["K"], seed)}
    M = case["M"]
    if op == "linear":
        N, K = case["N"], case["K"]
        act = inputs.activation_bf16 if fmt == "bf16" else inputs.activation
        need = P.fp6_linear_fgq_workspace_bytes(M, N, K, case["block"]) if fmt == "fgq" else _WORKSPACE[fmt](M, N, K)
        return {"case": case, "planes": _packed(case, N, K, seed), "X": act(M, K, seed + 1, device="cuda"),
                "Y": torch.empty((M, N), dtype=torch.bfloat16 if fmt == "bf16" else torch.float16, device="cuda"),
                "workspace": _zeros(need)}
    shapes = _block_shapes(case)
    h, kv, mlp = case["hidden"], case["kv"], case["mlp"]
    X = {"attn": inputs.activation(M, h, seed + 1, device="cuda"), "o": inputs.activation(M, h, seed + 2, device="cuda"),
         "mlp": inputs.activation(M, h, seed + 3, device="cuda"), "down": inputs.activation(M, mlp, seed + 4, device="cuda")}
    x_of = {"q": "attn", "k": "attn", "v": "attn", "o": "o", "gate": "mlp", "up": "mlp", "down": "down"}
    layer, Y = {}, {}
    for i, (name, N, K) in enumerate(shapes):
        layer[name] = (X[x_of[name]],) + tuple(_packed(case, N, K, seed + 10 + i)) + (N, K)
        Y[name] = torch.empty((M, N), dtype=torch.float16, device="cuda")
    need = max(P.fp6_linear_group_workspace_bytes(M, [(h, h), (kv, h), (kv, h)]), P.fp6_linear_workspace_bytes(M, h, h),
               P.fp6_linear_group_workspace_bytes(M, [(mlp, h), (mlp, h)]), P.fp6_linear_workspace_bytes(M, h, mlp))
    return {"case": case, "layer": layer, "Y": Y, "workspace": _zeros(need)}


def run(state):
    case = state["case"]
    op, fmt = case["op"], case["fmt"]
    if op == "quantize":
        return P.fp6_quantize_pack_fgq(state["W"], case["block"]) if fmt == "fgq" else _QUANTIZE[fmt](state["W"])
    if op == "dequantize":
        hi, lo, scales = state["planes"]
        if fmt == "fgq":
            return P.fp6_dequantize_fgq(hi, lo, scales, case["N"], case["K"], case["block"])
        return _DEQUANTIZE[fmt](hi, lo, scales, case["N"], case["K"])
    if op == "linear":
        hi, lo, scales = state["planes"]
        if fmt == "fgq":
            return P.fp6_linear_fgq(state["X"], hi, lo, scales, case["N"], case["K"], case["block"], out=state["Y"],
                                    workspace=state["workspace"])
        return _LINEAR[fmt](state["X"], hi, lo, scales, case["N"], case["K"], out=state["Y"], workspace=state["workspace"])
    L, Y, ws = state["layer"], state["Y"], state["workspace"]
    P.fp6_linear_group([L["q"], L["k"], L["v"]], outs=[Y["q"], Y["k"], Y["v"]], workspace=ws)
    P.fp6_linear(*L["o"], out=Y["o"], workspace=ws)
    P.fp6_linear_group([L["gate"], L["up"]], outs=[Y["gate"], Y["up"]], workspace=ws)
    P.fp6_linear(*L["down"], out=Y["down"], workspace=ws)
    return Y


def work(case):
    fmt = case["fmt"]

    def planes(N, K):
        per_row = K // case["block"] if fmt == "fgq" else 1
        return _PLANE_BYTES[fmt] * N * K + 2 * N * per_row

    if case["op"] in ("quantize", "dequantize"):
        N, K = case["N"], case["K"]
        return {"bytes": 2 * N * K + planes(N, K), "flops": 0}
    M = case["M"]
    if case["op"] == "linear":
        shapes, x_values = [(case["N"], case["K"])], M * case["K"]
    else:
        shapes = [(N, K) for _, N, K in _block_shapes(case)]
        x_values = M * (3 * case["hidden"] + case["mlp"])
    return {"bytes": sum(planes(N, K) + 2 * M * N for N, K in shapes) + 2 * x_values,
            "flops": sum(2 * M * N * K for N, K in shapes)}


def tolerance(case):
    # The offline step and its inverse are defined bit for bit.  A linear layer differs from its sum in 64 bits by
    # the rounding of the result to fp16 or bf16 (2-norm 2.1e-4 and 1.7e-3, largest 2^-11 and 2^-8), and by less than
    # that where only the order of its fp32 sums changes.
    if case["op"] in ("quantize", "dequantize"):
        return "exact"
    return {"rel": 7e-3, "max": 1.6e-2} if case["fmt"] == "bf16" else {"rel": 8e-4, "max": 2e-3}
