"""GPU parity of the paper-literal variant (float zero point, binary16, bias) against its
oracle: bit-exact materialization, forward / input-gradient / adapter-gradient outputs at
the stated bar and at a tight bound derived from the arithmetic."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from gpu_util import REL_LINF, assert_bar, f64
from oracle import paper_literal as pl
from paper_2309_16119_amd import binding as b
from paper_2309_16119_amd import synth

pytestmark = pytest.mark.gpu


def f16_dev(bits_u16):
    return torch.from_numpy(np.ascontiguousarray(bits_u16).view(np.int16)).cuda().view(torch.float16)


def layer(bits, K, N, M, r, group, seed=5, with_bias=True):
    cfg = synth.LayerConfig("t", K, N, bits, group, M, r, seed=seed)
    L = synth.make_layer_f16(cfg, with_bias=with_bias)
    D = dict(L)
    D["w"] = b.QWeightF16.from_numpy(L["qweight"], L["scales"], L["zeros_f16"], L["bias"], K, N, bits, group)
    D["Xd"], D["dYd"] = f16_dev(L["X"]), f16_dev(L["dY"])
    D["Ad"] = torch.from_numpy(L["A"]).cuda() if r else None
    D["Bd"] = torch.from_numpy(L["B"]).cuda() if r else None
    return D


def oargs(L):
    return (L["qweight"], L["scales"], L["zeros_f16"], L["K"], L["N"], L["bits"], L["group"])


def tight(name, got, ref, n_sum, out_f16=True, extra=0.0):
    """One binary16 rounding of the output (2^-11 relative) plus fp32 accumulation over n_sum terms."""
    scale = np.abs(ref).max()
    tol = (2.0 ** -10 if out_f16 else 2.0 ** -20) * np.abs(ref) + (4e-7 * np.sqrt(n_sum) + 2e-5) * scale + extra
    bad = np.abs(got - ref) > tol
    assert not bad.any(), "%s: %d elements off, worst %g (scale %g)" % (name, int(bad.sum()), float(np.abs(got - ref).max()), scale)


@pytest.mark.parametrize("bits,K,N,group", [(4, 256, 264, 64), (3, 1120, 808, 160), (2, 512, 520, 512), (3, 4096, 4096, 128)])
def test_dequant_bit_exact(bits, K, N, group):
    D = layer(bits, K, N, 1, 0, group)
    got = b.modulora_f16_dequant(D["w"]).view(torch.int16).cpu().numpy().view(np.uint16)
    ref = pl.dequant_f16(*oargs(D))
    assert np.array_equal(got, ref)


SHAPES = [
    # bits, K, N, M, r, group, bias
    (4, 256, 256, 16, 8, 64, True),
    (3, 1120, 808, 7, 3, 160, True),
    (2, 1088, 520, 33, 16, 64, False),
    (4, 544, 1304, 130, 40, 32, True),
    (3, 736, 776, 300, 64, 736, True),       # one (scale, zero) pair per row, maximum rank
    (2, 512, 2056, 515, 5, 128, True),
    (4, 2048, 512, 64, 0, 128, True),        # no adapter
    (3, 4096, 4096, 512, 8, 128, True),      # the headline shape
    # 128 tiles of 128 x 64 or more: the producer / consumer kernel, with a ragged row tile, ragged
    # column tiles and a ragged last 128-deep step in both directions
    (3, 2848, 2776, 300, 8, 32, True),
    (4, 2816, 2776, 300, 16, 2816, False),   # one (scale, zero) pair per row
    (2, 2944, 2752, 260, 40, 64, True),
    # about fifty 256 x 256 tiles in both directions: the 256 x 256 kernel with every tile cut into
    # slices of the contraction, whose partial tiles a second launch adds (ragged M and N)
    (3, 2816, 2456, 1100, 8, 128, True),
    (4, 2816, 2456, 1100, 0, 64, False),
    # a hundred-odd tokens (or that many past a multiple of 256) against a weight of 4096 x 4096 or more:
    # the kernel for up to 1024 tokens (ragged M, N, last step); the 256-column kernel with 128-row tiles,
    # which takes such token counts where that one does not, has a test of its own below
    (3, 4096, 4104, 100, 8, 128, True),
    (4, 4128, 4096, 128, 16, 32, False),
    (2, 4096, 4224, 300, 40, 64, True),
    # contractions shorter than one 64-deep step of the plain tile kernel (d_in = 32 forward, d_out = 48
    # backward) and outputs narrower than its tile: every load of the absent part stays inside its matrix
    (2, 32, 1664, 16, 0, 32, False),
    (4, 512, 48, 2, 8, 64, True),
    (2, 192, 96, 324, 33, 64, True),
    (3, 5632, 80, 12, 33, 5632, True),
]


# M <= 16 with shapes the streaming kernels accept: forward only (ragged last column block, group
# sizes down to one step), forward and backward (N and group multiples of 128), and N split over
# workgroups whose waves get unequal numbers of steps
STREAM_SHAPES = [
    (3, 4096, 4096, 17, 8, 128, True),       # 17 .. 32 tokens over more than 4 MB of codes: two passes
    (4, 2560, 4096, 32, 16, 64, False),
    (3, 1024, 808, 16, 8, 128, True),
    (3, 2560, 264, 3, 5, 256, False),
    (2, 768, 296, 5, 4, 64, True),
    (2, 1024, 1032, 16, 16, 128, True),
    (4, 512, 1304, 1, 16, 32, True),
    (4, 1152, 520, 13, 40, 128, False),
    (3, 1536, 512, 9, 0, 1536, True),        # one (scale, zero) pair per row, no adapter
    (3, 1024, 768, 16, 8, 128, True),
    (3, 2560, 384, 3, 5, 256, True),
    (2, 1024, 1152, 5, 16, 256, False),
    (4, 1152, 640, 13, 40, 128, True),
    (4, 512, 2304, 1, 16, 512, True),
    (2, 768, 128, 16, 0, 768, False),
    (2, 768, 384, 5, 4, 64, True),           # two quantization groups per 128-column backward tile
    (3, 1024, 2176, 11, 8, 64, False),
    (4, 512, 640, 16, 16, 64, True),
    (3, 1024, 2176, 11, 8, 128, True),
    (4, 512, 2176, 16, 4, 128, True),
    (2, 1024, 2176, 2, 8, 256, True),
]


def code_domain_allowance(D, M):
    """What the streaming kernels (M <= 32) may differ by from materialize-then-multiply: they multiply
    by the codes directly, so What is not rounded to binary16 first (2^-11 relative per weight), and
    the backward kernel rounds dY * scale to binary16 (another 2^-11 per term; a product below the
    normal range keeps 2^-25 absolute)."""
    if M > 32:
        return 0.0, 0.0
    Wabs = np.abs(synth.f16_bits_to_f64(pl.dequant_f16(*oargs(D))))          # [N][K]
    Xabs, dYabs = np.abs(synth.f16_bits_to_f64(D["X"])), np.abs(synth.f16_bits_to_f64(D["dY"]))
    qmax = float((1 << D["bits"]) - 1)
    return 2.0 ** -11 * (Xabs @ Wabs.T), 2.0 ** -10 * (dYabs @ Wabs) + 2.0 ** -25 * qmax * D["N"]


@pytest.mark.parametrize("bits,K,N,M,r,group,bias", SHAPES + STREAM_SHAPES)
def test_forward_backward_against_oracle(bits, K, N, M, r, group, bias):
    D = layer(bits, K, N, M, r, group, with_bias=bias)
    s = D["lora_scale"]
    A, B = (D["A"], D["B"]) if r else (None, None)
    Y, XA = b.modulora_f16_fwd(D["w"], D["Xd"], D["Ad"], D["Bd"], s)
    dX, T = b.modulora_f16_bwd_input(D["w"], D["dYd"], D["Ad"], D["Bd"], s)
    Yr, XAr = pl.fwd(*oargs(D), D["X"], A, B, s, D["bias"])
    dXr, Tr = pl.bwd_input(*oargs(D), D["dY"], A, B, s)
    extra_Y, extra_dX = code_domain_allowance(D, M)
    assert_bar("Y", f64(Y), Yr)
    assert_bar("dX", f64(dX), dXr)
    tight("Y", f64(Y), Yr, K + r, extra=extra_Y)
    tight("dX", f64(dX), dXr, N + r, extra=extra_dX)
    if r:
        tight("XA", f64(XA), XAr, K, out_f16=False)
        tight("dYBt", f64(T), Tr, N, out_f16=False)
        dA, dB = b.modulora_f16_bwd_lora(D["Xd"], D["dYd"], D["Ad"], D["Bd"], s, XA=XA, dYBt=T)
        dAr, dBr = pl.bwd_lora(D["X"], D["dY"], A, B, s)
        assert_bar("dA", f64(dA), dAr)
        assert_bar("dB", f64(dB), dBr)
        tight("dA", f64(dA), dAr, M + N, out_f16=False)
        tight("dB", f64(dB), dBr, M + K, out_f16=False)
        # the projections are recomputed when not handed over, and the accumulate flag adds
        dA2, dB2 = b.modulora_f16_bwd_lora(D["Xd"], D["dYd"], D["Ad"], D["Bd"], s, dA=dA.clone(), dB=dB.clone(), accumulate=True)
        tight("dA acc", f64(dA2), 2 * dAr, M + N, out_f16=False)
        tight("dB acc", f64(dB2), 2 * dBr, M + K, out_f16=False)


def test_one_hot_activations_pick_out_single_weights():
    """A one-hot row makes an output equal one What element (plus bias / nothing): bit for bit."""
    D = layer(3, 256, 264, 1, 0, 128, with_bias=False)
    What = pl.dequant_f16(*oargs(D))
    eyeK = torch.eye(256, dtype=torch.float16, device="cuda")
    Y, _ = b.modulora_f16_fwd(D["w"], eyeK[37:46].contiguous(), None, None, 1.0)
    assert np.array_equal(Y.view(torch.int16).cpu().numpy().view(np.uint16), What.T[37:46])
    eyeN = torch.eye(264, dtype=torch.float16, device="cuda")
    dX, _ = b.modulora_f16_bwd_input(D["w"], eyeN[100:101].contiguous(), None, None, 1.0)
    assert np.array_equal(dX.view(torch.int16).cpu().numpy().view(np.uint16), What[100:101])


def test_streaming_shapes_run_the_streaming_kernels():
    """The M <= 16 shapes above do reach the streaming kernels (in both directions where N and the
    group size allow)."""
    for K, N, M, passes in ((1024, 768, 16, 1), (4096, 4096, 20, 2)):
        D = layer(3, K, N, M, 8, 128)
        b.modulora_profile_begin()
        b.modulora_f16_fwd(D["w"], D["Xd"], D["Ad"], D["Bd"], 2.0)
        b.modulora_f16_bwd_input(D["w"], D["dYd"], D["Ad"], D["Bd"], 2.0)
        torch.cuda.synchronize()
        prof = b.modulora_profile_end()
        assert {k: v[0] for k, v in prof.items()} == {k: passes for k in ("f16_stream_fwd", "f16_stream_fwd_finish", "f16_stream_bwd",
                                                                          "f16_stream_bwd_finish")}, prof


@pytest.mark.parametrize("group", [128, 64])
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_streaming_kernels_pick_out_single_weights(bits, group):
    """One-hot rows through the M <= 16 streaming kernels: a single nonzero term, so the direct
    product with the codes must land on the same binary16 as the materialized weight -- in both
    directions (a one-hot 1.0 times the scale is the scale itself, so nothing is rounded early)."""
    K, N = 512, 384
    D = layer(bits, K, N, 1, 0, group, seed=6, with_bias=False)
    What = pl.dequant_f16(*oargs(D))
    eyeK = torch.eye(K, dtype=torch.float16, device="cuda")
    for lo in (0, 100, 497):
        Y, _ = b.modulora_f16_fwd(D["w"], eyeK[lo:lo + 15].contiguous(), None, None, 1.0)
        assert np.array_equal(Y.view(torch.int16).cpu().numpy().view(np.uint16), What.T[lo:lo + 15])
    eyeN = torch.eye(N, dtype=torch.float16, device="cuda")
    for lo in (0, 368):
        dX, _ = b.modulora_f16_bwd_input(D["w"], eyeN[lo:lo + 16].contiguous(), None, None, 1.0)
        assert np.array_equal(dX.view(torch.int16).cpu().numpy().view(np.uint16), What[lo:lo + 16])


def test_full_size_attention_projection_at_sixteen_tokens():
    """LLaMA-65B attention projection (8192 x 8192, 3-bit, group 128) at M = 16 in the paper's storage
    convention: the streaming kernels in the launch configuration of the full-size layer."""
    cfg = synth.CONFIGS["c5_65b_attn"].with_M(16)
    L = synth.make_layer_f16(cfg)
    w = b.QWeightF16.from_numpy(L["qweight"], L["scales"], L["zeros_f16"], L["bias"], cfg.K, cfg.N, cfg.bits, cfg.group)
    Xd, dYd = f16_dev(L["X"]), f16_dev(L["dY"])
    Ad, Bd = torch.from_numpy(L["A"]).cuda(), torch.from_numpy(L["B"]).cuda()
    s = L["lora_scale"]
    b.modulora_profile_begin()
    Y, XA = b.modulora_f16_fwd(w, Xd, Ad, Bd, s)
    dX, T = b.modulora_f16_bwd_input(w, dYd, Ad, Bd, s)
    torch.cuda.synchronize()
    assert {"f16_stream_fwd", "f16_stream_bwd"} <= set(b.modulora_profile_end())
    Yr, XAr = pl.fwd(*oargs(L), L["X"], L["A"], L["B"], s, L["bias"])
    dXr, Tr = pl.bwd_input(*oargs(L), L["dY"], L["A"], L["B"], s)
    extra_Y, extra_dX = code_domain_allowance(L, 16)
    assert_bar("Y", f64(Y), Yr)
    assert_bar("dX", f64(dX), dXr)
    tight("Y", f64(Y), Yr, cfg.K + cfg.r, extra=extra_Y)
    tight("dX", f64(dX), dXr, cfg.N + cfg.r, extra=extra_dX)
    tight("XA", f64(XA), XAr, cfg.K, out_f16=False)
    tight("dYBt", f64(T), Tr, cfg.N, out_f16=False)
    dA, dB = b.modulora_f16_bwd_lora(Xd, dYd, Ad, Bd, s, XA=XA, dYBt=T)
    dAr, dBr = pl.bwd_lora(L["X"], L["dY"], L["A"], L["B"], s)
    tight("dA", f64(dA), dAr, 16 + cfg.N, out_f16=False)
    tight("dB", f64(dB), dBr, 16 + cfg.K, out_f16=False)


def test_one_hot_activations_through_the_producer_consumer_kernel():
    """The same observation of the dequantization inside the kernel at a size that takes the
    128 x 64 producer / consumer kernel (300 one-hot rows, 132 tiles in both directions)."""
    K, N = 2816, 2776
    D = layer(3, K, N, 1, 0, 128, with_bias=False)
    What = pl.dequant_f16(*oargs(D))
    eyeK = torch.eye(K, dtype=torch.float16, device="cuda")
    Y, _ = b.modulora_f16_fwd(D["w"], eyeK[100:400].contiguous(), None, None, 1.0)
    assert np.array_equal(Y.view(torch.int16).cpu().numpy().view(np.uint16), What.T[100:400])
    eyeN = torch.eye(N, dtype=torch.float16, device="cuda")
    dX, _ = b.modulora_f16_bwd_input(D["w"], eyeN[200:500].contiguous(), None, None, 1.0)
    assert np.array_equal(dX.view(torch.int16).cpu().numpy().view(np.uint16), What[200:500])


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_large_shape_on_sampled_rows_and_one_hot(bits):
    """Close to 200 tiles of 256 x 256 in both directions: the 256 x 256 kernel's binary16
    instantiation (ragged last row tile).  The oracle's cost is linear in the token count, so Y
    and dX are checked on sampled token rows (a row of Y / dX depends only on the same row of
    X / dY); one-hot activations make the dequantization inside the kernel observable bit for bit."""
    K, N, M, r, group = 4096, 3584, 3500, 8, 128
    D = layer(bits, K, N, M, r, group, seed=9, with_bias=True)
    s = D["lora_scale"]
    Y, XA = b.modulora_f16_fwd(D["w"], D["Xd"], D["Ad"], D["Bd"], s)
    dX, T = b.modulora_f16_bwd_input(D["w"], D["dYd"], D["Ad"], D["Bd"], s)
    rows = np.unique(np.concatenate(([0, M - 1, 3327, 3328], np.random.default_rng(3).integers(0, M, 8))))
    Yr, XAr = pl.fwd(*oargs(D), np.ascontiguousarray(D["X"][rows]), D["A"], D["B"], s, D["bias"])
    dXr, Tr = pl.bwd_input(*oargs(D), np.ascontiguousarray(D["dY"][rows]), D["A"], D["B"], s)
    assert_bar("Y", f64(Y)[rows], Yr)
    assert_bar("dX", f64(dX)[rows], dXr)
    tight("Y", f64(Y)[rows], Yr, K + r)
    tight("dX", f64(dX)[rows], dXr, N + r)
    tight("XA", f64(XA)[rows], XAr, K, out_f16=False)
    tight("dYBt", f64(T)[rows], Tr, N, out_f16=False)

    E = layer(bits, K, N, 1, 0, group, seed=9, with_bias=False)
    What = pl.dequant_f16(*oargs(E))
    eyeK = torch.eye(K, dtype=torch.float16, device="cuda")
    Y1, _ = b.modulora_f16_fwd(E["w"], eyeK[300:300 + M].contiguous(), None, None, 1.0)
    assert np.array_equal(Y1.view(torch.int16).cpu().numpy().view(np.uint16), What.T[300:300 + M])
    del eyeK, Y1
    eyeN = torch.eye(N, dtype=torch.float16, device="cuda")
    dX1, _ = b.modulora_f16_bwd_input(E["w"], eyeN[:M].contiguous(), None, None, 1.0)
    assert np.array_equal(dX1.view(torch.int16).cpu().numpy().view(np.uint16), What[:M])


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_half_row_tiles_of_the_256_column_kernel(bits):
    """Token counts whose last block of 256 rows is at most half full, past what the kernel for up to 1024
    tokens takes: the 128-row instantiation of the 256-column kernel (the producer / consumer and the plain
    kernel have no second launch, and 256-row tiles are not chosen at five blocks of 128 rows), ragged in
    rows, columns and the last step of both contractions; sampled rows, and one-hot rows bit for bit."""
    K, N, M, r, group = 4128, 4104, 520, 16, 96
    D = layer(bits, K, N, M, r, group, seed=15)
    s = D["lora_scale"]
    b.modulora_profile_begin()
    Y, XA = b.modulora_f16_fwd(D["w"], D["Xd"], D["Ad"], D["Bd"], s)
    dX, T = b.modulora_f16_bwd_input(D["w"], D["dYd"], D["Ad"], D["Bd"], s)
    torch.cuda.synchronize()
    names = {k for k in b.modulora_profile_end() if not k.startswith("lora_")}
    assert names == {"f16_gemm_fwd", "f16_gemm_fwd_fixup", "f16_gemm_bwd", "f16_gemm_bwd_fixup"}, names
    rows = np.unique(np.concatenate(([0, 127, 128, 383, 511, 512, M - 1], np.random.default_rng(3).integers(0, M, 40))))
    Yr, XAr = pl.fwd(*oargs(D), np.ascontiguousarray(D["X"][rows]), D["A"], D["B"], s, D["bias"])
    dXr, Tr = pl.bwd_input(*oargs(D), np.ascontiguousarray(D["dY"][rows]), D["A"], D["B"], s)
    tight("Y", f64(Y)[rows], Yr, K + r)
    tight("dX", f64(dX)[rows], dXr, N + r)
    tight("XA", f64(XA)[rows], XAr, K, out_f16=False)
    tight("dYBt", f64(T)[rows], Tr, N, out_f16=False)

    E = layer(bits, K, N, 1, 0, group, seed=15, with_bias=False)
    What = b.modulora_f16_dequant(E["w"])            # [N][K], bit-exact against the oracle (above)
    for lo in (0, K - M):
        X = torch.zeros((M, K), dtype=torch.float16, device="cuda")
        X[torch.arange(M), lo + torch.arange(M)] = 1.0
        Y1, _ = b.modulora_f16_fwd(E["w"], X, None, None, 1.0)
        assert torch.equal(Y1.view(torch.int16), What.t()[lo:lo + M].contiguous().view(torch.int16))
    for lo in (0, N - M):
        dY = torch.zeros((M, N), dtype=torch.float16, device="cuda")
        dY[torch.arange(M), lo + torch.arange(M)] = 1.0
        dX1, _ = b.modulora_f16_bwd_input(E["w"], dY, None, None, 1.0)
        assert torch.equal(dX1.view(torch.int16), What[lo:lo + M].contiguous().view(torch.int16))


def test_outputs_do_not_depend_on_stale_memory():
    D = layer(4, 512, 520, 40, 8, 64)
    s = D["lora_scale"]
    Y0, _ = b.modulora_f16_fwd(D["w"], D["Xd"], D["Ad"], D["Bd"], s)
    Y1 = torch.full_like(Y0, float("nan"))
    b._workspaces.clear()
    b.modulora_f16_fwd(D["w"], D["Xd"], D["Ad"], D["Bd"], s, Y=Y1)
    assert torch.equal(Y0.view(torch.int16), Y1.view(torch.int16))


def test_operands_beyond_four_gib():
    """A million tokens: X, dY, Y and dX are 4.5 GB each, so rows past index 2^20 lie beyond
    4 GiB from the start of their matrices.  A few thousand rows, spread over the range and
    dense at its end, are populated; the others are zero, so their outputs must be exactly the
    bias (Y) or zero (dX), and the sums over tokens reduce to the populated rows, which is all
    the oracle is given."""
    K = N = 2048
    bits, group, r = 3, 128, 8
    M = (1 << 20) + (1 << 16) + 3
    rng = np.random.default_rng(9)
    live = np.unique(np.concatenate((rng.integers(0, M, 3800), np.arange(M - 150, M), [0, 1 << 20, (1 << 20) + 1])))
    n_live = live.size
    D = layer(bits, K, N, n_live, r, group, seed=13, with_bias=True)
    s = D["lora_scale"]
    live_t = torch.from_numpy(live).cuda()
    X = torch.zeros((M, K), dtype=torch.float16, device="cuda")
    dY = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    X[live_t] = D["Xd"]
    dY[live_t] = D["dYd"]
    assert int(live[-1]) * K * 2 > (1 << 32)

    Y, XA = b.modulora_f16_fwd(D["w"], X, D["Ad"], D["Bd"], s)
    dX, T = b.modulora_f16_bwd_input(D["w"], dY, D["Ad"], D["Bd"], s)
    dA, dB = b.modulora_f16_bwd_lora(X, dY, D["Ad"], D["Bd"], s, XA=XA, dYBt=T)
    torch.cuda.synchronize()

    is_live = torch.zeros(M, dtype=torch.bool, device="cuda")
    is_live[live_t] = True
    bias_d = f16_dev(D["bias"])
    assert torch.equal(Y.ne(bias_d).any(dim=1), is_live), "Y"
    for name, out in (("dX", dX), ("XA", XA), ("dYBt", T)):
        assert torch.equal(out.ne(0).any(dim=1), is_live), name

    pick = np.unique(np.concatenate((np.arange(n_live - 24, n_live), rng.integers(0, n_live, 24))))
    pick_t = live_t[torch.from_numpy(pick).cuda()]
    Yr, XAr = pl.fwd(*oargs(D), np.ascontiguousarray(D["X"][pick]), D["A"], D["B"], s, D["bias"])
    dXr, Tr = pl.bwd_input(*oargs(D), np.ascontiguousarray(D["dY"][pick]), D["A"], D["B"], s)
    assert_bar("Y", f64(Y[pick_t]), Yr)
    assert_bar("dX", f64(dX[pick_t]), dXr)
    tight("Y", f64(Y[pick_t]), Yr, K + r)
    tight("dX", f64(dX[pick_t]), dXr, N + r)
    tight("XA", f64(XA[pick_t]), XAr, K, out_f16=False)
    tight("dYBt", f64(T[pick_t]), Tr, N, out_f16=False)
    dAr, dBr = pl.bwd_lora(D["X"], D["dY"], D["A"], D["B"], s)
    assert_bar("dA", f64(dA), dAr)
    assert_bar("dB", f64(dB), dBr)
    tight("dA", f64(dA), dAr, n_live * N, out_f16=False)
    tight("dB", f64(dB), dBr, n_live * K, out_f16=False)


@pytest.mark.parametrize("K,N,M,r,bits", [
    (544, 264, 17, 3, 3),            # one ragged tile, an extension that ends inside a step
    (1120, 2056, 130, 64, 4),        # 128 x 64 tiles, three steps of 128 and more for the extension
    (2816, 2456, 1100, 33, 2),       # 256 x 256 tiles cut into slices, the last of which takes the extension
    (96, 4104, 2100, 16, 3),         # whole 256 x 256 tiles whose extension is as long as the contraction
])
def test_adapter_term_through_the_extended_contraction(K, N, M, r, bits):
    """An adapter term thirty times the base product, whose six-segment split has to carry what fp32 does:
    the error against float64 stays within the output's rounding (2^-11) plus that of fp32 sums.  An
    infinite factor gives the infinities of the definition and NaN nowhere else."""
    D = layer(bits, K, N, M, r, 32, seed=21)
    A, B, s = D["A"] * np.float32(30), D["B"] * np.float32(30), D["lora_scale"]
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = np.unique(np.concatenate(([0, M - 1, M // 2], np.random.default_rng(2).integers(0, M, 20))))
    Y, _ = b.modulora_f16_fwd(D["w"], D["Xd"], Ad, Bd, s)
    dX, _ = b.modulora_f16_bwd_input(D["w"], D["dYd"], Ad, Bd, s)
    Yr, _ = pl.fwd(*oargs(D), np.ascontiguousarray(D["X"][rows]), A, B, s, D["bias"])
    dXr, _ = pl.bwd_input(*oargs(D), np.ascontiguousarray(D["dY"][rows]), A, B, s)
    for got, ref, n in ((f64(Y)[rows], Yr, K + r), (f64(dX)[rows], dXr, N + r)):
        assert np.all(np.abs(got - ref) <= 2.0 ** -11 * np.abs(ref) + 6e-8 * np.sqrt(n) * np.abs(ref).max() + 2.0 ** -25)
    Bi = Bd.clone()
    Bi[r - 1, 5] = float("inf")
    Ai = Ad.clone()
    Ai[7, r - 1] = -float("inf")
    Y2, _ = b.modulora_f16_fwd(D["w"], D["Xd"], Ad, Bi, s)
    dX2, _ = b.modulora_f16_bwd_input(D["w"], D["dYd"], Ai, Bd, s)
    for got, was, col in ((Y2, Y, 5), (dX2, dX, 7)):
        assert bool(torch.isinf(got[:, col]).all())
        keep = torch.arange(got.shape[1], device="cuda") != col
        assert torch.equal(got[:, keep].view(torch.int16), was[:, keep].view(torch.int16))


@pytest.mark.parametrize("bits,K,N,M,r,fwd", [
    (4, 256, 384, 9, 8, "single"),           # the projection beside the one-launch product
    (2, 896, 2176, 15, 33, "single"),        # ... with three groups of rank columns, the last of one
    (4, 4096, 4096, 16, 8, "stream"),        # sixteen projecting workgroups, the streaming kernels' own second launch
    (3, 4096, 4224, 27, 5, "stream"),        # two passes, the second of eleven rows
    (3, 512, 1152, 16, 64, "stream"),        # the shared second launch
])
def test_infinite_activations_in_the_projection_of_few_tokens(bits, K, N, M, r, fwd):
    """X A and dY B^T of an infinite activation (an overflow, no rarity in binary16) or factor: the infinities that the
    definition gives, NaN only where one meets zero or its opposite, every other element as without them."""
    D = layer(bits, K, N, M, r, 128 if K % 256 == 0 and bits == 3 else 64, seed=13)
    inf, nan = float("inf"), float("nan")
    for backward, act, F in ((False, D["Xd"].clone(), D["Ad"].clone()), (True, D["dYd"].clone(), D["Bd"].t().contiguous())):
        C = act.shape[1]
        act[0, 5], act[1, 3], act[1, 9] = inf, inf, -inf
        act[M - 1, C - 1], act[2, C // 2] = -inf, nan
        act[M - 2, 17] = 0.0
        F[5, r // 2] = 0.0                                   # meets the infinity of row 0
        F[17, r - 1] = -inf                                  # meets the zero of row M - 2
        A, B = (F, D["Bd"]) if not backward else (D["Ad"], F.t().contiguous())
        call = b.modulora_f16_bwd_input if backward else b.modulora_f16_fwd
        b.modulora_profile_begin()
        _, P = call(D["w"], act, A, B, 2.0)
        torch.cuda.synchronize()
        names = set(b.modulora_profile_end())
        want = {"f16_stream_bwd", "f16_stream_bwd_finish"} if backward else \
               {"f16_stream_fwd_single"} if fwd == "single" else {"f16_stream_fwd", "f16_stream_fwd_finish"}
        assert names == want
        for j in range(r):
            terms = act.double() * F[:, j].double()
            ref, mag, got = terms.sum(1), terms.abs().sum(1), P[:, j].double()
            assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isposinf(), ref.isposinf()) and torch.equal(got.isneginf(), ref.isneginf())
            ok = ref.isfinite()
            assert bool(((got - ref).abs()[ok] <= (2.0 ** -24 * (64 + C ** 0.5) * mag)[ok]).all())


@pytest.mark.parametrize("backward", [False, True])
def test_extended_contraction_is_as_exact_as_fp32(backward):
    """One product p f per output (rank 1, one-hot rows, a weight of zeros), carried as six segments: the output is the
    product's own binary16 rounding wherever the product lies further than 2^-22 of itself from a rounding boundary
    (2^-24 that the segments leave out, 2^-23 for the matrix cores' sum of the six).  The operands stand just above a power of
    two with long runs of ones, where a split is at its worst: a split by truncation misses by up to 2^-21 there,
    and a hundred outputs and more land on the wrong side of the boundary."""
    K, N = 1056, 4104
    rng = np.random.default_rng(4)

    def factor(n):               # 1.0000000 11xxxxxx 1xxxxxxx
        low = 0xC080 | (rng.integers(0, 64, n, dtype=np.uint32) << 8) | rng.integers(0, 128, n, dtype=np.uint32)
        return (np.uint32(0x3F800000) | low.astype(np.uint32)).view(np.float32)
    A, B = factor(K).reshape(K, 1), factor(N).reshape(1, N)
    w = b.QWeightF16(torch.zeros((K // 8, N), dtype=torch.int32, device="cuda"), torch.zeros((K // 32, N), dtype=torch.float16, device="cuda"),
                     torch.zeros((K // 32, N), dtype=torch.float16, device="cuda"), None, K, N, 4, 32)
    act = torch.eye(K, N if backward else K, dtype=torch.float16, device="cuda")
    call = b.modulora_f16_bwd_input if backward else b.modulora_f16_fwd
    b.modulora_profile_begin()
    out, P = call(w, act, torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), 1.0)
    torch.cuda.synchronize()
    assert "lora_down" in b.modulora_profile_end()           # the tile kernels, which take the segments
    p, f = (B[0, :K], A[:, 0]) if backward else (A[:, 0], B[0])
    assert np.array_equal(P[:, 0].cpu().numpy(), p)
    exact = np.multiply.outer(p.astype(np.float64), f.astype(np.float64))
    half = exact.astype(np.float16)
    boundary = np.abs(np.abs(exact - half.astype(np.float64)) - np.spacing(half).astype(np.float64) / 2)
    got = out.cpu().numpy()
    assert int(((got != half) & (boundary > 2.0 ** -22 * exact)).sum()) == 0


PLAIN = """
import torch
from paper_2309_16119_amd import binding as b, synth
for bits, K, N, M, r in ((3, 544, 264, 33, 3), (4, 1024, 2056, 300, 64), (2, 256, 512, 20, 0)):
    L = synth.make_layer_torch(synth.LayerConfig("t", K, N, bits, 32, M, max(r, 1)), device="cuda", seed=3)
    bias = torch.randn(N, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).half()
    w = b.QWeightF16(L["qweight"], L["scales"], -2 * L["scales"], bias, K, N, bits, 32)
    W = b.modulora_f16_dequant(w).double()
    X, dY, A, B = L["X"].half(), L["dY"].half(), *((L["A"] * 3, L["B"] * 30) if r else (None, None))
    b.modulora_profile_begin()
    Y, _ = b.modulora_f16_fwd(w, X, A, B, 2.0)
    dX, _ = b.modulora_f16_bwd_input(w, dY, A, B, 2.0)
    torch.cuda.synchronize()
    assert {k for k in b.modulora_profile_end() if not k.startswith("lora_")} == {"f16_gemm_fwd", "f16_gemm_bwd"}
    Yr, dXr, mY, mX = X.double() @ W.t() + bias.double(), dY.double() @ W, X.double().abs() @ W.abs().t(), dY.double().abs() @ W.abs()
    if r:
        A, B = A.double(), B.double()
        Yr, dXr = Yr + 2 * (X.double() @ A) @ B, dXr + 2 * (dY.double() @ B.t()) @ A.t()
        mY, mX = mY + 2 * (X.double().abs() @ A.abs()) @ B.abs(), mX + 2 * (dY.double().abs() @ B.abs().t()) @ A.abs().t()
    for got, ref, mag, n in ((Y, Yr, mY, K), (dX, dXr, mX, N)):      # one rounding, fp32 sums
        assert bool(((got.double() - ref).abs() <= 2.0 ** -11 * ref.abs() + 2.0 ** -24 * (64 + n ** 0.5) * mag + 2.0 ** -25).all())
print("plain kernel agrees")
"""


def test_plain_kernel_for_comparisons():
    """MODULORA_F16_PLAIN, read once per process: every shape that no streaming kernel takes on the plain kernel."""
    res = subprocess.run([sys.executable, "-c", PLAIN], capture_output=True, text=True, timeout=100,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), env={**os.environ, "MODULORA_F16_PLAIN": "1"})
    assert res.returncode == 0 and "plain kernel agrees" in res.stdout, res.stdout + res.stderr[-2000:]
