"""What a user of this framework has it do, as cases that can be timed and compared.

A case names one operation of the public Python interface and its sizes:

  op "fwd"       one modulora_fwd / modulora_f16_fwd call (serving: no hand-off for a backward pass)
  op "step"      forward, input gradient and adapter gradients of one layer through the three library
                 calls, with the hand-offs XA and dYBt between them (one layer's share of a training step)
  op "module"    the same through nn.ModuLoRALinear and autograd
  op "quantize"  modulora_quantize_rtn of a float32 weight (what prepares a layer)

`kind` is "bf16" (integer zero points, bfloat16 activations) or "f16" (the paper's own storage
convention: added binary16 zero points, binary16 activations, a bias).  K = d_in, N = d_out, M tokens,
r the adapter's rank, g the group size.  Values are those of the layers that synth.CONFIGS describes.
"""
from __future__ import annotations

import math

import torch

from paper_2309_16119_amd import binding, nn, synth

LORA_SCALE = 2.0


def _case(name, op, K, N, bits, g, M, r, kind="bf16"):
    return {"name": name, "op": op, "kind": kind, "K": K, "N": N, "bits": bits, "g": g, "M": M, "r": r}


def listed():
    return [
        # A layer so small that only launches and the host path count.
        _case("step_256_m16", "step", 256, 256, 4, 64, 16, 8),
        # Generating one token: every linear layer reads its whole packed weight for one row.
        _case("decode_7b_gate_m1", "fwd", 4096, 11008, 4, 128, 1, 16),
        # Generating a batch of tokens with the largest matrix of a 65B layer.
        _case("decode_65b_up_m16", "fwd", 8192, 22016, 3, 128, 16, 8),
        # Training on a very short sample, both directions: still a stream over the packed weight.
        _case("step_65b_down_m16", "step", 22016, 8192, 3, 128, 16, 8),
        # A short prompt: too many rows for one matrix-core tile, far too few to be bound by arithmetic.
        _case("step_65b_attn_m48", "step", 8192, 8192, 3, 128, 48, 8),
        # One sequence of 512 tokens through an attention projection of the 7B model.
        _case("step_7b_attn_m512", "step", 4096, 4096, 3, 128, 512, 8),
        # The same in the paper's own storage convention.
        _case("f16_step_7b_attn_m512", "step", 4096, 4096, 3, 128, 512, 8, "f16"),
        # Sequences of real text have no round length: a ragged batch through the autograd module.
        _case("module_7b_down_m777", "module", 11008, 4096, 4, 128, 777, 16),
        # 1024 tokens through a 2-bit attention projection of the 30B model, two groups per 128 inputs.
        _case("step_30b_attn_m1024", "step", 6656, 6656, 2, 64, 1024, 8),
        # A batch of four sequences of 512 tokens through the 7B model's MLP, 4 bits.
        _case("step_7b_gate_m2048", "step", 4096, 11008, 4, 128, 2048, 16),
        # The largest: 4096 tokens through the 65B model's widest matrix.
        _case("step_65b_up_m4096", "step", 8192, 22016, 3, 128, 4096, 8),
        # Quantizing that matrix.
        _case("quantize_65b_up", "quantize", 8192, 22016, 3, 128, 0, 0),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(["fwd", "fwd", "step", "step", "step", "module", "quantize"])
    kind = "f16" if op != "quantize" and rng.random() < 0.25 else "bf16"
    bits = rng.choice([2, 3, 4])
    g = rng.choice([64, 128, 128, 128])
    # Widths of real layers are multiples of 128; some are not.
    unit_k, unit_n = (128, 128) if rng.random() < 0.75 else (g, rng.choice([8, 32, 64]))
    K = max(256, int(_log_uniform(rng, 256, 22016)) // unit_k * unit_k)
    N = max(256, int(_log_uniform(rng, 256, 22016)) // unit_n * unit_n)
    if K * N > 8192 * 22016:
        K = max(256, 8192 * 22016 // N // unit_k * unit_k)
    if op == "quantize":
        return {"op": op, "kind": kind, "K": K, "N": N, "bits": bits, "g": g, "M": 0, "r": 0}
    M = int(round(_log_uniform(rng, 1, 4096)))
    r = rng.choice([8, 8, 8, 16, 16, 4, 32, 64] + ([0] if op == "fwd" else []))
    return {"op": op, "kind": kind, "K": K, "N": N, "bits": bits, "g": g, "M": M, "r": r}


def _config(case):
    scale = (0.01, 0.04) if case["bits"] == 2 else (0.005, 0.02)
    return synth.LayerConfig("case", case["K"], case["N"], case["bits"], case["g"], max(case["M"], 1), case["r"],
                             scale[0], scale[1], LORA_SCALE)


def prepare(case, seed):
    K, N, M, r = case["K"], case["N"], case["M"], case["r"]
    state = dict(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["op"] == "quantize":
        state["W"] = torch.randn((N, K), device="cuda", generator=gen) * 0.02
        return state
    cfg = _config(case)
    layer = synth.make_layer_torch(cfg, device="cuda", seed=seed)
    shape = (K, N, case["bits"], case["g"])
    if case["kind"] == "f16":
        span = ((1 << case["bits"]) - 1) * cfg.scale_hi
        zeros = (torch.rand((K // case["g"], N), device="cuda", generator=gen) * -span).to(torch.float16)
        bias = (torch.randn(N, device="cuda", generator=gen) * 0.1).to(torch.float16)
        w = binding.QWeightF16(layer["qweight"], layer["scales"], zeros, bias, *shape)
        dtype = torch.float16
    else:
        w = binding.QWeight(layer["qweight"], layer["scales"], layer["zeros"], *shape)
        dtype = torch.bfloat16
    state["w"] = w
    state["X"], state["dY"] = layer["X"].to(dtype), layer["dY"].to(dtype)
    state["A"], state["B"] = (layer["A"], layer["B"]) if r else (None, None)
    if case["op"] == "module":
        module = nn.ModuLoRALinear(w, r=r, alpha=LORA_SCALE * r)
        with torch.no_grad():
            module.A.copy_(layer["A"])
            module.B.copy_(layer["B"])
        state["module"] = module
        state["X"].requires_grad_(True)
    return state


def run(state):
    op = state["op"]
    if op == "quantize":
        w = binding.modulora_quantize_rtn(state["W"], state["bits"], state["g"])
        return w.qweight, w.scales, w.zeros
    w, X, dY, A, B = state["w"], state["X"], state["dY"], state["A"], state["B"]
    if op == "module":
        module = state["module"]
        Y = module(X)
        dX, dA, dB = torch.autograd.grad(Y, (X, module.A, module.B), dY)
        return Y.detach(), dX, dA, dB
    if state["kind"] == "f16":
        fwd, bwd_input, bwd_lora = binding.modulora_f16_fwd, binding.modulora_f16_bwd_input, binding.modulora_f16_bwd_lora
    else:
        fwd, bwd_input, bwd_lora = binding.modulora_fwd, binding.modulora_bwd_input, binding.modulora_bwd_lora
    if op == "fwd":
        return fwd(w, X, A, B, LORA_SCALE, want_XA=False)[0]
    Y, XA = fwd(w, X, A, B, LORA_SCALE)
    dX, dYBt = bwd_input(w, dY, A, B, LORA_SCALE)
    dA, dB = bwd_lora(X, dY, A, B, LORA_SCALE, XA=XA, dYBt=dYBt)
    return Y, XA, dX, dYBt, dA, dB


def work(case):
    K, N, M, r = case["K"], case["N"], case["M"], case["r"]
    packed = K * N * case["bits"] / 8 + K // case["g"] * N * (4 if case["kind"] == "f16" else 3)
    if case["op"] == "quantize":
        return {"bytes": 4 * K * N + packed, "flops": 0}
    adapter = 4 * r * (K + N)
    if case["op"] == "fwd":
        return {"bytes": packed + 2 * M * (K + N) + adapter, "flops": 2 * M * K * N + 2 * M * r * (K + N)}
    # A model's forward and backward passes lie a whole model apart: each reads the frozen weight.
    return {"bytes": 2 * packed + 4 * M * (K + N) + 2 * adapter, "flops": 4 * M * K * N + 6 * M * r * (K + N)}


def tolerance(case):
    # Against the same path in 64 bits: rel 1.7e-3 where What is materialized (the one rounding of the
    # result), 2.3e-3 to 2.9e-3 with at most 1.2e-2 off where the codes are multiplied directly; in
    # binary16 an eighth of that.  Stated is about four times as much.
    if case["op"] == "quantize":
        return "exact"
    if case["kind"] == "f16":
        return {"rel": 1.5e-3, "max": 1e-2}
    return {"rel": 1e-2, "max": 5e-2}
