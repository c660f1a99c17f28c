"""The adapter-gradient kernel where its tiles end: 32-row blocks, 64- and 128-column blocks, groups
of 16 adapter columns, waves without rows, row chunks with the reduction launch; both activation
types, with and without accumulation, against float64 products of the same operands."""
import numpy as np
import pytest
import torch

from paper_2309_16119_amd import binding as b, synth

pytestmark = pytest.mark.gpu

SHAPES = [
    # K, N, M, r
    (32, 8, 1, 1),
    (64, 72, 31, 16),
    (96, 136, 33, 17),
    (128, 64, 64, 48),
    (160, 200, 515, 33),           # 16 waves, most of them with one block more than the others
    (96, 264, 300, 64),
    (64, 40, 1030, 3),             # one row chunk: too few rows for two
    (256, 264, 2051, 8),           # two row chunks and the reduction launch
    (64, 128, 4200, 40),
    (8192, 8456, 4100, 8),         # from 128 MB of activations on: eight columns per lane
    (16384, 264, 4105, 20),
    (4096, 4232, 2900, 8),         # binary16: eight columns per lane, three chunks
    (8192, 8456, 300, 16),         # binary16: eight columns per lane below 128 MB
    (8192, 8456, 256, 16),         # four
    (8192, 8456, 6200, 3),         # three or more chunks of 131 column blocks
    (4096, 4232, 4100, 40),        # the same at 131 blocks of 64 columns
]


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("K,N,M,r", SHAPES)
def test_adapter_gradients_at_tile_edges(K, N, M, r, f16):
    gen = torch.Generator(device="cuda").manual_seed(K + 3 * N + M)
    dtype = torch.float16 if f16 else torch.bfloat16
    X = torch.randn((M, K), device="cuda", generator=gen).to(dtype)
    dY = torch.randn((M, N), device="cuda", generator=gen).to(dtype)
    XA = torch.randn((M, r), device="cuda", generator=gen)
    T = torch.randn((M, r), device="cuda", generator=gen)
    A, B = torch.zeros((K, r), device="cuda"), torch.zeros((r, N), device="cuda")
    s = 0.75
    call = b.modulora_f16_bwd_lora if f16 else b.modulora_bwd_lora
    dA = torch.full((K, r), float("nan"), device="cuda")
    dB = torch.full((r, N), float("nan"), device="cuda")
    call(X, dY, A, B, s, XA=XA, dYBt=T, dA=dA, dB=dB)
    dA0 = torch.randn((K, r), device="cuda", generator=gen)
    dB0 = torch.randn((r, N), device="cuda", generator=gen)
    dA2, dB2 = dA0.clone(), dB0.clone()
    call(X, dY, A, B, s, XA=XA, dYBt=T, dA=dA2, dB=dB2, accumulate=True)
    # fp32 sums of M exact products: the rounding errors of M additions, taken as independent, times 8
    unit = 8 * np.sqrt(M) * 2.0 ** -24 * s
    for got, got2, old, act, P, left in ((dA, dA2, dA0, X, T, True), (dB, dB2, dB0, dY, XA, False)):
        a64, p64 = act.double(), P.double()
        ref = s * (a64.T @ p64 if left else p64.T @ a64)
        mag = a64.abs().T @ p64.abs() if left else p64.abs().T @ a64.abs()
        assert bool(((got.double() - ref).abs() <= unit * mag + 1e-30).all())
        assert bool(((got2.double() - ref - old.double()).abs() <= unit * mag + 2.0 ** -23 * (ref + old.double()).abs() + 1e-30).all())


@pytest.mark.parametrize("K,N,M,r,f16", [(8192, 8320, 8192, 8, False), (8192, 8320, 4096, 8, True), (4096, 4232, 4100, 64, False)])
def test_rows_are_cut_where_column_blocks_fill_half_the_chip(K, N, M, r, f16):
    """129 ... 131 column blocks on 256 compute units: one chunk of rows would leave half of them idle."""
    dtype = torch.float16 if f16 else torch.bfloat16
    X, dY = torch.zeros((M, K), dtype=dtype, device="cuda"), torch.zeros((M, N), dtype=dtype, device="cuda")
    P = torch.zeros((M, r), device="cuda")
    A, B = torch.zeros((K, r), device="cuda"), torch.zeros((r, N), device="cuda")
    b.modulora_profile_begin()
    (b.modulora_f16_bwd_lora if f16 else b.modulora_bwd_lora)(X, dY, A, B, 1.0, XA=P, dYBt=P)
    torch.cuda.synchronize()
    assert {k: v[0] for k, v in b.modulora_profile_end().items()} == {"lora_grad": 1, "lora_grad_reduce": 1}


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("K,N,M,r", [(64, 72, 31, 16), (96, 136, 600, 17), (160, 264, 70, 64), (8192, 8264, 300, 8)])
def test_infinities_stay_infinities(K, N, M, r, f16):
    """Overflowed activations or hand-offs (common in binary16): an infinite factor gives +-inf in the sums
    that it enters and NaN only where it meets zero or an opposite infinity, and leaves the others alone."""
    gen = torch.Generator(device="cuda").manual_seed(M)
    dtype = torch.float16 if f16 else torch.bfloat16
    X, dY = (torch.randn((M, c), device="cuda", generator=gen).to(dtype) for c in (K, N))
    XA, T = (torch.randint(1, 9, (M, r), device="cuda", generator=gen).float() / 4 for _ in range(2))   # exact in bfloat16
    X[M // 2, 3], X[M - 1, K - 1], X[0, 8] = float("inf"), float("-inf"), float("nan")
    dY[M // 3, 5] = float("-inf")
    dY[0, 11] = dY[M - 1, 11] = float("inf")
    T[M // 4, r // 2], XA[1, 0] = float("inf"), float("-inf")
    X[M // 4, 9], dY[1, 7] = 0.0, 0.0
    A, B = torch.zeros((K, r), device="cuda"), torch.zeros((r, N), device="cuda")
    dA, dB = (b.modulora_f16_bwd_lora if f16 else b.modulora_bwd_lora)(X, dY, A, B, 0.5, XA=XA, dYBt=T)
    for got, act, P, left in ((dA, X, T, True), (dB, dY, XA, False)):
        for j in range(r):
            terms = 0.5 * act.double() * P[:, j:j + 1].double()
            ref, mag = terms.sum(0), terms.abs().sum(0)
            g = (got[:, j] if left else got[j]).double()
            assert torch.equal(g.isnan(), ref.isnan()) and torch.equal(g.isposinf(), ref.isposinf()) and torch.equal(g.isneginf(), ref.isneginf())
            ok = ref.isfinite()
            assert bool(((g - ref).abs()[ok] <= (8 * np.sqrt(M) * 2.0 ** -24 * mag + 1e-30)[ok]).all())


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("M,K,N,r", [
    (256, 2048, 2056, 33),      # the smallest by tiles; B^T: the last chunk of 128 holds eight elements
    (321, 2144, 4104, 64),      # a wave with one row, contractions that end inside a chunk
    (1029, 4128, 6152, 17),     # rank over 16
    (1025, 6176, 6280, 5),      # a rank that is no multiple of four, one row past the last block
])
def test_projections_by_tiles(M, K, N, r, f16):
    """X A and dY B^T of the forward and backward calls by tiles (rows and ranks past lora_down_plan()'s line),
    against float64: fp32 products (the split is exact) summed in fp32; and the adapter term that is
    built from them, through the outputs of a layer whose weight is zero."""
    gen = torch.Generator(device="cuda").manual_seed(M)
    dtype = torch.float16 if f16 else torch.bfloat16
    X = torch.randn((M, K), device="cuda", generator=gen).to(dtype)
    dY = torch.randn((M, N), device="cuda", generator=gen).to(dtype)
    A = torch.randn((K, r), device="cuda", generator=gen) * 0.02
    B = torch.randn((r, N), device="cuda", generator=gen) * 0.02
    words = torch.zeros((K * 3 // 32, N), dtype=torch.int32, device="cuda")
    scales = torch.ones((K // 32, N), dtype=torch.float16, device="cuda")
    if f16:
        w = b.QWeightF16(words, scales, torch.zeros_like(scales), None, K, N, 3, 32)
        fwd, bwd, rounding = b.modulora_f16_fwd, b.modulora_f16_bwd_input, 2.0 ** -11
    else:
        w = b.QWeight(words, scales, torch.zeros((K // 32, N), dtype=torch.uint8, device="cuda"), K, N, 3, 32)
        fwd, bwd, rounding = b.modulora_fwd, b.modulora_bwd_input, 2.0 ** -8
    Y, XA = fwd(w, X, A, B, 2.0)
    dX, T = bwd(w, dY, A, B, 2.0)
    P, Q = X.double() @ A.double(), dY.double() @ B.double().t()
    # 32 units of 2^-24 of the sum of absolute products: fp32 sums of up to 64 steps per slice, then the slices
    errs = []
    for got, ref, act, F in ((XA, P, X, A), (T, Q, dY, B.t())):
        bound = (act.double().abs() @ F.double().abs()) * 2.0 ** -24 * 32 + 2.0 ** -20 * ref.abs()
        assert bool(((got.double() - ref).abs() <= bound).all()), float((got.double() - ref).abs().max())
        errs.append(bound)
    # the projection's error times the other factor, the split of the extended contraction, one rounding
    for got, proj, err, F in ((Y, P, errs[0], B.double()), (dX, Q, errs[1], A.double().t())):
        ref = 2.0 * proj @ F
        bound = rounding * ref.abs() + 2.0 * (err + (2.0 ** -20 if f16 else 2.0 ** -15) * proj.abs()) @ F.abs() + 2.0 ** -25
        assert bool(((got.double() - ref).abs() <= bound).all()), float((got.double() - ref).abs().max())


@pytest.mark.parametrize("K,N,M,r,backward", [
    (4128, 4440, 303, 64, True),      # by tiles since the estimates choose, in fp32 before
    (1056, 4104, 130, 3, False),
    (1056, 4104, 2200, 17, False),
])
def test_infinite_factor_through_the_extended_contraction(K, N, M, r, backward):
    """bfloat16 tile kernels: an infinite adapter factor gives infinities in its output column, NaN where it meets zeros
    only, and leaves every other column as it was."""
    cfg = synth.LayerConfig("t", K, N, 3, 32, M, r)
    L = synth.make_layer_torch(cfg, device="cuda", seed=17)
    w = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, 3, 32)
    A, B = L["A"].clone(), L["B"].clone()
    act, call = (L["dY"], b.modulora_bwd_input) if backward else (L["X"], b.modulora_fwd)
    act[3] = 0.0                                              # projects to zeros
    was, P = call(w, act, A, B, 2.0)
    F = A if backward else B.t()
    F[5, r - 1], F[9, 0] = float("inf"), -float("inf")
    b.modulora_profile_begin()
    got, P2 = call(w, act, A, B, 2.0)
    torch.cuda.synchronize()
    assert "lora_down" in b.modulora_profile_end()            # the tile kernels
    assert torch.equal(P, P2)
    for col, j, sign in ((5, r - 1, 1.0), (9, 0, -1.0)):
        assert torch.equal(got[:, col].double().nan_to_num(0.0, 1.0, -1.0), torch.sign(P[:, j].double()) * sign)
        assert bool(got[3, col].isnan()) and not bool(got[:3, col].isnan().any())
    keep = torch.ones(got.shape[1], dtype=torch.bool, device="cuda")
    keep[5] = keep[9] = False
    assert torch.equal(got[:, keep].view(torch.int16), was[:, keep].view(torch.int16))
