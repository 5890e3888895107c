"""Workloads whose run time matters to a program that uses this library, as cases that can be measured.

A case is a dict of plain values.  Its `kind` says which calls one pass makes:

  layer   the seven linears of one decoder layer from fp32 activations, as four calls of `mpgemm_f32` (q|k|v and gate|up
          stacked along M with one weight scale per row, o, down), outputs and workspaces held by the caller: what a
          serving loop runs per layer and step, from one decoded token to a long prefill
  f32     one linear from fp32 activations: `mpgemm_f32`, which allocates its output and workspace like any torch op
  codes   `quantize_act` once, then `mpgemm` for each of `reuse` matrices that share the input (the two-call form)
  g5      as codes, on the 1.60-bit packing (`mpgemm_g5`; K a multiple of 20)
  mixed   as codes, on the mixed 1.60-bit / 2-bit packing (`mpgemm_mixed`; any K that 4 divides)
  pack    ternary weights to the packed blob (`pack_weights` or `pack_weights_mixed`): once per matrix at model load

Shapes are those of `paper_2512_06443_amd.workloads` (2B, 3B and 8B shaped linears, 1 to 1024 tokens) or generic.
"""
from __future__ import annotations

import math

import torch

from paper_2512_06443_amd import binding as B

# Linears of one 2.4B-style decoder layer, stacked where they share their input: name -> (rows of each matrix, K).
LAYER = (("qkv", (2560, 640, 640), 2560), ("o", (2560,), 2560), ("gateup", (6912, 6912), 2560), ("down", (2560,), 6912))
W_SIGMA = 0.02                      # latent weights are N(0, W_SIGMA^2); their mean magnitude is the weight scale
W_SCALE = W_SIGMA * math.sqrt(2.0 / math.pi)


def _case(name, kind, M=0, K=0, N=0, p_zero=0.4, outliers=0.0, acc=False, reuse=1, mixed=False):
    return {"name": name, "kind": kind, "M": M, "K": K, "N": N, "p_zero": p_zero, "outliers": outliers, "acc": acc,
            "reuse": reuse, "mixed": mixed}


def listed():
    return [
        # the smallest call: a 256 x 256 matrix and eight tokens; latency of one call and its launches
        _case("tiny_n8", "f32", 256, 256, 8, p_zero=1.0 / 3.0),
        # decoding one sequence: every weight of the layer is streamed for a single token
        _case("layer_n1", "layer", N=1),
        # batched decoding or speculative verification: a few sequences at once
        _case("layer_n16", "layer", N=16),
        # a short prompt or a large decoding batch
        _case("layer_n64", "layer", N=64),
        # a long prompt in one piece
        _case("layer_n1024", "layer", N=1024),
        # three projections of one input in the two-call form, a handful of tokens
        _case("kv_codes_n4", "codes", 640, 2560, 4, reuse=3),
        # the FFN up projection on a 128-token prompt, two-call form
        _case("ffn_up_codes_n128", "codes", 6912, 2560, 128),
        # odd sizes and the raw accumulators: rows, features and tokens that no tile divides
        _case("ragged_acc_n77", "f32", 3203, 3116, 77, acc=True),
        # the largest matrix on a 512-token prompt, activations with outlier channels
        _case("gateup8b_n512", "f32", 14336, 4096, 512, p_zero=0.35, outliers=0.01),
        # long rows: few output rows for the work, K = 14336
        _case("down8b_n512", "f32", 4096, 14336, 512, p_zero=0.35, outliers=0.01),
        # the smaller packing where memory is what counts: K that 5 does not divide, batched decoding
        _case("mixed_qo8b_n32", "mixed", 4096, 4096, 32, p_zero=0.35),
        # model load: one large matrix from ternary bytes to the blob
        _case("pack8b", "pack", 14336, 4096, p_zero=0.35),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "f32", "f32", "f32", "codes", "codes", "g5", "mixed", "pack"])
    p_zero = rng.choice([1.0 / 3.0, 0.35, 0.4])
    outliers = rng.choice([0.0, 0.01])
    if kind == "layer":
        return _case("", kind, N=_log_int(rng, 1, 1024), p_zero=p_zero, outliers=outliers)
    M, K = _log_int(rng, 200, 14336), _log_int(rng, 256, 14336)
    if rng.random() < 0.5:          # half of the matrices with sizes that models have: multiples of 128
        M, K = max(128, M // 128 * 128), max(256, K // 128 * 128)
    K = K // 20 * 20 if kind == "g5" else K // 4 * 4
    # the 1.60-bit packings are for decoding and short prompts; no case above the work of the largest listed one
    cap = 14336 * 4096 * 512 // (4 if kind in ("g5", "mixed") else 1)
    N = min(_log_int(rng, 1, 256 if kind in ("g5", "mixed") else 1024), max(1, cap // (M * K)))
    if kind == "pack":
        return _case("", kind, M, K, p_zero=p_zero, mixed=rng.random() < 0.3)
    reuse = rng.choice([1, 3]) if kind == "codes" and M * K * N < cap // 4 else 1
    return _case("", kind, M, K, N, p_zero, outliers, acc=rng.random() < 0.25, reuse=reuse)


def _weights(gen, M, K, p_zero):
    u = torch.rand((M, K), generator=gen, device="cuda")
    p_neg = 0.5 * (1.0 - p_zero)
    return (u >= p_neg).to(torch.int8) + (u >= p_neg + p_zero).to(torch.int8) - 1


def _activations(gen, N, K, outliers):
    x = torch.randn((N, K), generator=gen, device="cuda")
    if outliers > 0.0:
        ch = torch.randperm(K, generator=gen, device="cuda")[:math.ceil(outliers * K)]
        x[:, ch] *= 20.0
    return x


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, N = case["kind"], case["N"]
    if kind == "layer":
        lib = B.lib()
        calls = []
        for i, (_, rows, K) in enumerate(LAYER):
            M = sum(rows)
            packed = B.pack_weights(_weights(gen, M, K, case["p_zero"]))
            scale = W_SCALE
            if len(rows) > 1:       # stacked matrices: each row carries its own matrix' scale
                scale = torch.cat([torch.full((m,), W_SCALE * (1.0 + 0.1 * j), device="cuda") for j, m in enumerate(rows)])
            x = _activations(gen, N, K, case["outliers"])
            y = torch.empty((N, M), dtype=torch.float32, device="cuda")
            ws = torch.empty(max(lib.vlut_workspace_bytes_f32(M, K, N), 16), dtype=torch.uint8, device="cuda")
            calls.append((packed, scale, x, M, y, ws))
        return {"kind": kind, "calls": calls}
    M, K = case["M"], case["K"]
    state = {"kind": kind, "M": M, "acc": case["acc"], "mixed": case["mixed"]}
    if kind == "pack":
        state["w"] = _weights(gen, M, K, case["p_zero"])
        return state
    pack = {"f32": B.pack_weights, "codes": B.pack_weights, "g5": B.pack_weights_g5, "mixed": B.pack_weights_mixed}[kind]
    state["packed"] = [pack(_weights(gen, M, K, case["p_zero"])) for _ in range(case["reuse"])]
    state["x"] = _activations(gen, N, K, case["outliers"])
    return state


def run(state):
    kind = state["kind"]
    if kind == "layer":
        for packed, scale, x, M, y, ws in state["calls"]:
            B.mpgemm_f32(packed, scale, x, M, y=y, workspace=ws)
        return [call[4] for call in state["calls"]]
    if kind == "pack":
        return (B.pack_weights_mixed if state["mixed"] else B.pack_weights)(state["w"])
    M, acc = state["M"], state["acc"]
    if kind == "f32":
        y, a, scales = B.mpgemm_f32(state["packed"][0], W_SCALE, state["x"], M, want_acc=acc, want_scales=acc)
        return [y, a, scales] if acc else [y]
    mpgemm = {"codes": B.mpgemm, "g5": B.mpgemm_g5, "mixed": B.mpgemm_mixed}[kind]
    a_q, a_scale = B.quantize_act(state["x"])
    out = [a_q, a_scale]
    for packed in state["packed"]:
        y, a = mpgemm(packed, W_SCALE, a_q, a_scale, M, want_acc=acc)
        out += [y, a] if acc else [y]
    return out


def _blob_bytes(kind, M, K, mixed=False):
    groups = {"g5": K // 5, "mixed": K // 20 * 4 + (K - K // 20 * 20) // 4}
    return M * (groups["mixed"] if mixed else groups.get(kind, K // 4))


def work(case):
    """Bytes and operations of one pass: packed weights, activations, codes where the caller sees them, and outputs once
    each; a multiply and an add per weight and token."""
    kind, N = case["kind"], case["N"]
    if kind == "layer":
        mats = [(sum(rows), K, 4 * sum(rows) if len(rows) > 1 else 0) for _, rows, K in LAYER]
        return {"bytes": sum(M * K // 4 + scales + 4 * N * K + 4 * N * M for M, K, scales in mats),
                "flops": sum(2 * M * K * N for M, K, _ in mats)}
    M, K = case["M"], case["K"]
    if kind == "pack":
        return {"bytes": M * K + _blob_bytes(kind, M, K, case["mixed"]), "flops": 0}
    out = N * M * (8 if case["acc"] else 4)
    if kind == "f32":
        return {"bytes": M * K // 4 + 4 * N * K + out + (4 * N if case["acc"] else 0), "flops": 2 * M * K * N}
    codes = (N + 7) // 8 * 8 * K + 4 * N
    return {"bytes": 4 * N * K + codes + case["reuse"] * (_blob_bytes(kind, M, K) + out), "flops": case["reuse"] * 2 * M * K * N}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    # Codes, scales and accumulators are whole numbers or decided in fp32: equal.  An output is a whole number below
    # 2^24 times two fp32 scales: two roundings.  Against the same product in 64 bits that is 3.5e-8 in the 2-norm and
    # 1.1e-7 for the worst value; four times that is what another correct implementation may show.
    return {"rel": 1.5e-7, "max": 4.5e-7}
