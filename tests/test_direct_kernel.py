"""The kernel for a few dozen to a thousand tokens (gemm_direct.hip) where it can go wrong: row blocks of
one to four tiles of 32 rows and more than one block, outputs that end inside a column block, contractions
that end inside a chunk of 256, a step of 64 or a half of one, groups of one 32-code block up to the whole
row, every rank class, slices; both directions, both storage conventions, against the two oracles."""
import os
import re
import subprocess

import numpy as np
import pytest
import torch

import oracle
from oracle import paper_literal as pl
from paper_2309_16119_amd import binding as b
from paper_2309_16119_amd import build, synth

from test_kernel_resources import _hipcc

# bits, d_in, d_out, tokens, rank, group
SHAPES = [
    (3, 4096, 2056, 33, 8, 128),        # two row tiles; backward contraction ends 8 elements into a chunk
    (4, 4256, 4104, 65, 17, 224),       # three row tiles; forward contraction ends in half a step
    (2, 2080, 4104, 100, 5, 32),        # four row tiles; a group per 32-code block
    (3, 4160, 4104, 129, 64, 4160),     # two row blocks; one group per row
    (4, 4128, 2304, 256, 16, 96),       # odd number of blocks per group
    (2, 4128, 8200, 100, 0, 32),        # no adapter
    (3, 4096, 4096, 512, 8, 128),       # four row blocks
    (4, 4096, 2568, 777, 8, 128),       # seven row blocks, the last ragged, whole contractions
    (2, 4000, 3336, 1000, 33, 4000),    # eight
    (3, 8224, 2624, 20, 8, 32),         # one row tile: a shape that no streaming kernel takes
    (4, 4096, 2104, 7, 33, 128),        # a handful of tokens that the backward streaming kernel does not take
    (3, 288, 32768, 40, 8, 288),        # an output of little more than two column blocks (backward only)
    # under 2^23 weights, an output of whole column blocks in both directions
    (3, 2432, 2944, 64, 8, 128),
    (4, 2560, 2560, 33, 16, 32),
    (2, 2688, 2304, 150, 3, 64),
    (3, 2944, 2432, 5, 8, 32),          # a handful of tokens, groups of 32 at three bits: no streaming kernel
    (2, 2048, 2176, 257, 33, 2048),     # three row blocks, one group per row
    (4, 3200, 2560, 20, 0, 128),        # no adapter, a weight too small for two streaming passes
]


def _ran(call, conv, direction):
    b.modulora_profile_begin()
    out = call()
    torch.cuda.synchronize()
    names = set(b.modulora_profile_end())
    return out, (("f16_gemm_" if conv == "f16" else "gemm_") + direction + "_direct") in names


def _close(got, ref, rel, n_sum):
    got = got.float().cpu().numpy().astype(np.float64)
    tol = rel * np.abs(ref) + (4e-7 * np.sqrt(n_sum) + 2e-5) * np.abs(ref).max()
    assert np.all(np.abs(got - ref) <= tol), float(np.abs(got - ref).max())


@pytest.mark.gpu
@pytest.mark.parametrize("conv", ["bf16", "f16"])
@pytest.mark.parametrize("bits,K,N,M,r,group", SHAPES)
def test_against_the_oracle(bits, K, N, M, r, group, conv):
    cfg = synth.LayerConfig("t", K, N, bits, group, M, r, seed=77)
    s, f16 = 2.0, conv == "f16"
    if f16:
        L = synth.make_layer_f16(cfg)
        w = b.QWeightF16.from_numpy(L["qweight"], L["scales"], L["zeros_f16"], L["bias"], K, N, bits, group)
        act = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda().view(torch.float16)
        oa = (L["qweight"], L["scales"], L["zeros_f16"], K, N, bits, group)
        fwd, bwd, rel = b.modulora_f16_fwd, b.modulora_f16_bwd_input, 2.0 ** -10
    else:
        L = synth.make_layer(cfg)
        w = b.QWeight.from_numpy(L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
        act = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda().view(torch.bfloat16)
        oa = (L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
        fwd, bwd, rel = b.modulora_fwd, b.modulora_bwd_input, 2.0 ** -8
    A, B = (L["A"], L["B"]) if r else (None, None)
    Ad, Bd = (torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()) if r else (None, None)
    X, dY = act(L["X"]), act(L["dY"])
    nan = lambda cols: torch.full((M, cols), float("nan"), dtype=X.dtype, device="cuda")
    (Y, XA), ran_fwd = _ran(lambda: fwd(w, X, Ad, Bd, s, nan(N)), conv, "fwd")
    (dX, T), ran_bwd = _ran(lambda: bwd(w, dY, Ad, Bd, s, nan(K)), conv, "bwd")
    assert ran_bwd and (ran_fwd or M < 16 or K < 512), (ran_fwd, ran_bwd)
    if f16:
        Yr, Ur = pl.fwd(*oa, L["X"], A, B, s, L["bias"])
        dXr, Tr = pl.bwd_input(*oa, L["dY"], A, B, s)
    else:
        Yr, Ur = oracle.fwd(*oa, L["X"], A, B, s)
        dXr, Tr = oracle.bwd_input(*oa, L["dY"], A, B, s)
    if ran_fwd:
        _close(Y, Yr, rel, K + r)
    _close(dX, dXr, rel, N + r)
    if r:
        _close(XA, Ur, 2.0 ** -20, K)
        _close(T, Tr, 2.0 ** -20, N)
    # no atomics: a second run gives the same bits
    assert torch.equal(dX.view(torch.int16), bwd(w, dY, Ad, Bd, s)[0].view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("conv", ["bf16", "f16"])
@pytest.mark.parametrize("bits,K,N,M,r,group", [
    # second launches of up to 16 rows behind the streaming kernels: 32, 64 and 128 columns a workgroup, ranks that
    # fill a group of 16 or not, that are no multiple of four, one row, sixteen, two passes
    (4, 512, 640, 1, 9, 128),
    (3, 2560, 384, 16, 64, 128),
    (2, 768, 16512, 5, 17, 64),
    (4, 512, 32896, 3, 33, 128),
    (3, 4096, 4096, 29, 16, 128),
    # sixteen tokens, which the one-launch kernel leaves to two launches: 32 columns a workgroup, 64 forward, 64 backward
    (4, 512, 640, 16, 9, 128),
    (2, 768, 16512, 16, 17, 64),
    (3, 16640, 512, 16, 17, 128),
    # and of 32 rows behind the direct kernel, deep and not: one row past a tile, a rank of 1, 2, 47 and 64
    (3, 4096, 2056, 33, 1, 128),
    (2, 4096, 4104, 65, 2, 32),
    (4, 4128, 2304, 63, 47, 96),
    (3, 4096, 4096, 700, 64, 128),
    (3, 4096, 4096, 545, 15, 128),
    # many workgroups and a rank of up to eight: a last row, last columns of eight, a rank that is no multiple of four,
    # one column of rank with seven slices (forward) and sixteen parts (backward), nine parts
    (3, 4096, 4104, 545, 8, 128),
    (4, 4128, 4096, 600, 3, 96),
    (2, 8192, 8200, 200, 1, 64),
    (3, 17920, 3336, 330, 5, 128),
])
def test_second_launch_adds_slices_and_adapter(bits, K, N, M, r, group, conv):
    """An adapter term that is most of the output (factors times thirty), so that a part, a slice or a column of
    the second launch that went missing or to the wrong place cannot hide."""
    cfg = synth.LayerConfig("t", K, N, bits, group, M, r, seed=78)
    s, f16 = 2.0, conv == "f16"
    if f16:
        L = synth.make_layer_f16(cfg)
        w = b.QWeightF16.from_numpy(L["qweight"], L["scales"], L["zeros_f16"], L["bias"], K, N, bits, group)
        What, dtype = b.modulora_f16_dequant(w), torch.float16
        fwd, bwd, rel = b.modulora_f16_fwd, b.modulora_f16_bwd_input, 2.0 ** -10
    else:
        L = synth.make_layer(cfg)
        w = b.QWeight.from_numpy(L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
        What, dtype = b.modulora_dequant(w), torch.bfloat16
        fwd, bwd, rel = b.modulora_fwd, b.modulora_bwd_input, 2.0 ** -8
    act = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda().view(dtype)
    X, dY, W = act(L["X"]), act(L["dY"]), What.double()
    A, B = torch.from_numpy(L["A"]).cuda() * 30, torch.from_numpy(L["B"]).cuda() * 30
    nan = lambda cols, t: torch.full((M, cols), float("nan"), dtype=t, device="cuda")
    b.modulora_profile_begin()
    Y, XA = fwd(w, X, A, B, s, nan(N, dtype), nan(r, torch.float32))
    dX, T = bwd(w, dY, A, B, s, nan(K, dtype), nan(r, torch.float32))
    torch.cuda.synchronize()
    names = set(b.modulora_profile_end())
    if M == 16:
        assert names == {("f16_" if f16 else "") + "stream_" + which for which in ("fwd", "fwd_finish", "bwd", "bwd_finish")}
    XAr, Tr = X.double() @ A.double(), dY.double() @ B.double().t()
    Yr = X.double() @ W.t() + s * XAr @ B.double()
    if f16:
        Yr = Yr + act(L["bias"]).double()
    dXr = dY.double() @ W + s * Tr @ A.double().t()
    # what multiplying by the codes instead of the rounded weight may change (up to 32 tokens)
    extra_Y = extra_dX = 0.0
    if M <= 32:
        unit = (2.0 ** -11 if f16 else 2.0 ** -8)
        extra_Y = (unit * X.double().abs() @ W.abs().t()).cpu().numpy()
        extra_dX = (2 * unit * dY.double().abs() @ W.abs()).cpu().numpy() + (2.0 ** -25 * 15 * N if f16 else 0.0)
    for got, ref, n, extra in ((Y, Yr, K + r, extra_Y), (dX, dXr, N + r, extra_dX)):
        got, ref = got.double().cpu().numpy(), ref.cpu().numpy()
        assert np.all(np.abs(got - ref) <= rel * np.abs(ref) + (4e-7 * np.sqrt(n) + 2e-5) * np.abs(ref).max() + extra)
    _close(XA, XAr.cpu().numpy(), 2.0 ** -20, K)
    _close(T, Tr.cpu().numpy(), 2.0 ** -20, N)


@pytest.mark.gpu
@pytest.mark.parametrize("conv,direction,K,N,M,r,direct", [
    # the rank's price: an output of 69 column blocks, whose 32 projection parts the second launch adds in a row
    ("bf16", "fwd", 1024, 8832, 38, 8, True),
    ("bf16", "fwd", 1024, 8832, 38, 64, False),
    ("bf16", "bwd", 9728, 1536, 288, 16, True),
    ("bf16", "bwd", 9728, 1536, 288, 32, False),
    # the tile kernels of binary16 pay for a rank as well
    ("f16", "fwd", 3072, 3072, 245, 64, True),
    ("bf16", "fwd", 4096, 4096, 129, 64, True),
    # five rounds of workgroups against whole 256-row tiles, three against 128-row ones (a last block of 88 rows)
    ("bf16", "fwd", 6656, 17920, 392, 8, False),
    ("f16", "fwd", 6656, 17920, 407, 8, False),
    ("bf16", "fwd", 22016, 8192, 600, 8, True),
    ("bf16", "fwd", 6656, 6656, 777, 8, True),
    # under 2^23 weights: by the estimate where the output is a whole number of column blocks
    ("bf16", "fwd", 3840, 1024, 40, 8, True),
    ("f16", "fwd", 2560, 2176, 35, 8, True),
    ("bf16", "bwd", 512, 11136, 143, 8, True),
    ("bf16", "fwd", 4096, 1064, 100, 8, False),
    ("bf16", "bwd", 1024, 256, 464, 16, False),     # few workgroups share the projection
    ("bf16", "fwd", 256, 1024, 64, 8, False),       # a contraction of one chunk
])
def test_runs_where_it_is_the_quicker_way(conv, direction, K, N, M, r, direct):
    cfg = synth.LayerConfig("t", K, N, 3, 128, M, r)
    L = synth.make_layer_torch(cfg, device="cuda", seed=9)
    act = L["X"] if direction == "fwd" else L["dY"]
    if conv == "f16":
        w = b.QWeightF16(L["qweight"], L["scales"], -L["scales"], None, K, N, 3, 128)
        call = b.modulora_f16_fwd if direction == "fwd" else b.modulora_f16_bwd_input
        act = act.to(torch.float16)
    else:
        w = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, 3, 128)
        call = b.modulora_fwd if direction == "fwd" else b.modulora_bwd_input
    assert _ran(lambda: call(w, act, L["A"], L["B"], 2.0), conv, direction)[1] == direct


@pytest.mark.gpu
@pytest.mark.parametrize("conv", ["bf16", "f16"])
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_picks_out_single_weights_bit_for_bit(bits, conv):
    """One-hot rows: an output is one materialized weight, in every lane and register position."""
    K, N, group, M = 4160, 4104, 32, 96
    f16 = conv == "f16"
    cfg = synth.LayerConfig("t", K, N, bits, group, 1, 0, seed=5)
    if f16:
        L = synth.make_layer_f16(cfg, with_bias=False)
        w = b.QWeightF16.from_numpy(L["qweight"], L["scales"], L["zeros_f16"], None, K, N, bits, group)
        What = b.modulora_f16_dequant(w)
        fwd, bwd, dtype = b.modulora_f16_fwd, b.modulora_f16_bwd_input, torch.float16
    else:
        L = synth.make_layer(cfg)
        w = b.QWeight.from_numpy(L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
        What = b.modulora_dequant(w)            # [N][K], bit-exact against the oracle (test_gpu_parity.py)
        fwd, bwd, dtype = b.modulora_fwd, b.modulora_bwd_input, torch.bfloat16
    for lo in (0, K // 2 - 48, K - M):
        rows = torch.zeros((M, K), dtype=dtype, device="cuda")
        rows[torch.arange(M), lo + torch.arange(M)] = 1.0
        (Y, _), ran = _ran(lambda: fwd(w, rows, None, None, 1.0), conv, "fwd")
        assert ran and torch.equal(Y.view(torch.int16), What.t()[lo:lo + M].contiguous().view(torch.int16))
    for lo in (0, N // 2 - 52, N - M):
        rows = torch.zeros((M, N), dtype=dtype, device="cuda")
        rows[torch.arange(M), lo + torch.arange(M)] = 1.0
        (dX, _), ran = _ran(lambda: bwd(w, rows, None, None, 1.0), conv, "bwd")
        assert ran and torch.equal(dX.view(torch.int16), What[lo:lo + M].contiguous().view(torch.int16))


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_kernels_do_not_spill(tmp_path):
    """The kernel counts its assembly-issued loads and keeps registers untouched while they are in flight."""
    out = tmp_path / "gemm_direct.s"
    cmd = [_hipcc(), *build.HIPCC_FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "gemm_direct.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    text = out.read_text()
    names = re.findall(r"^\s*\.name:\s+(\S+)", text, flags=re.M)
    assert sum("gemm_direct_kernel" in n for n in names) == 48     # 3 bit widths x 2 directions x 2 conventions x 4 row tiles
    spills = re.findall(r"^\s*\.[vs]gpr_spill_count:\s+(\d+)", text, flags=re.M)
    assert len(spills) == 2 * len(names) and all(int(s) == 0 for s in spills)
    assert "scratch_load" not in text and "scratch_store" not in text
