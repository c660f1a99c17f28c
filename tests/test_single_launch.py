"""A small layer's call in one launch (single.hip): either width of its workgroups, ranks that fill a
group of 16 or not, ragged rows and outputs, contractions of fewer units than waves and of several rounds.  Up to 15
tokens against the product with the unrounded weight in 64 bits, and against the two launches that sixteen take;
more tokens against the product with the rounded weight."""
import pytest
import torch

from paper_2309_16119_amd import binding as b, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("conv", ["bf16", "f16"])
@pytest.mark.parametrize("bits,K,N,M,r,group", [
    (4, 256, 256, 15, 8, 64),          # eight units: one per wave
    (3, 256, 488, 1, 0, 128),          # no adapter, a last workgroup of eight columns
    (2, 384, 264, 3, 9, 64),           # twelve units
    (4, 896, 2104, 7, 16, 32),         # a rank that fills its group, one step per quantization group
    (3, 896, 1032, 5, 17, 896),        # one group per row
    (2, 1024, 272, 13, 32, 128),       # two rounds of units in flight
    (4, 1920, 520, 2, 1, 384),         # a last round of half the waves
    (3, 256, 17032, 9, 8, 128),        # workgroups of 64 columns, the last of eight
    (2, 512, 12040, 4, 24, 64),
    (4, 256, 9608, 15, 47, 64),
])
def test_one_launch(bits, K, N, M, r, group, conv):
    cfg = synth.LayerConfig("t", K, N, bits, group, M, max(r, 1))
    L = synth.make_layer_torch(cfg, device="cuda", seed=29)
    f16 = conv == "f16"
    dtype, call = (torch.float16, b.modulora_f16_fwd) if f16 else (torch.bfloat16, b.modulora_fwd)
    words = (L["qweight"].long() & 0xFFFFFFFF).view(K // 32, bits, N)
    code = []
    for pos in range(0, 32 * bits, bits):               # the 32 codes of a block, two of which may straddle words
        v = words[:, pos // 32] >> (pos % 32)
        if pos % 32 + bits > 32:
            v = v | (words[:, pos // 32 + 1] << (32 - pos % 32))
        code.append(v & ((1 << bits) - 1))
    codes, s = torch.stack(code, dim=1).reshape(K, N).double(), L["scales"].double().repeat_interleave(group, dim=0)
    if f16:
        zeros = (L["zeros"].float() * -L["scales"].float()).half()
        bias = torch.randn(N, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).half()
        w, W = b.QWeightF16(L["qweight"], L["scales"], zeros, bias, K, N, bits, group), codes * s + zeros.double().repeat_interleave(group, dim=0)
    else:
        w, W = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, bits, group), (codes - L["zeros"].double().repeat_interleave(group, dim=0)) * s
    A, B = (L["A"] * 3, L["B"] * 30) if r else (None, None)      # an adapter term as large as the product
    X = torch.randn((16, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(2)).to(dtype)
    out = torch.full((M, N), float("nan"), dtype=dtype, device="cuda")
    b.modulora_profile_begin()
    Y, XA = call(w, X[:M].contiguous(), A, B, 2.0, out)
    torch.cuda.synchronize()
    assert set(b.modulora_profile_end()) == {("f16_" if f16 else "") + "stream_fwd_single"}
    X64 = X[:M].double()
    ref, mag = X64 @ W, X64.abs() @ (codes.abs() + (1088 if f16 else 136 + L["zeros"].double().repeat_interleave(group, dim=0))).mul(s)
    if r:
        down = X64 @ A.double()
        assert bool(((XA.double() - down).abs() <= 2.0 ** -24 * (64 + K ** 0.5) * (X64.abs() @ A.double().abs())).all())
        ref, mag = ref + 2 * down @ B.double(), mag + 2 * (X64.abs() @ A.double().abs()) @ B.double().abs()
    if f16:
        ref = ref + bias.double()
    # one rounding of the output; fp32 sums of products with the offset codes
    tol = (2.0 ** -11 if f16 else 2.0 ** -8) * ref.abs() + 2.0 ** -24 * (64 + K ** 0.5) * mag
    assert bool(((Y.double() - ref).abs() <= tol).all()), float(((Y.double() - ref).abs() / tol).max())
    # sixteen tokens take two launches: the same rows to the same accuracy
    both = call(w, X, A, B, 2.0)[0][:M].double()
    assert bool(((both - ref).abs() <= tol).all())


@pytest.mark.parametrize("conv", ["bf16", "f16"])
@pytest.mark.parametrize("bits,K,N,M,r,group", [
    (4, 256, 256, 17, 8, 64),          # two workgroups' rows, the second of one
    (3, 256, 496, 252, 4, 32),         # groups of one block, a last row block of 28
    (2, 384, 272, 33, 9, 64),
    (4, 896, 2064, 48, 16, 32),        # a rank that fills its group
    (3, 416, 1040, 100, 17, 416),      # one group per row, thirteen units
    (2, 768, 272, 131, 64, 128),
    (4, 1152, 528, 31, 1, 384),
    (3, 1088, 272, 20, 0, 64),         # no adapter, 34 units
    (3, 256, 5136, 70, 8, 128),        # workgroups of 64 columns, the last of 16
    (2, 512, 4112, 64, 32, 64),
    (4, 256, 7696, 40, 47, 64),
])
def test_one_launch_with_the_rounded_weight(bits, K, N, M, r, group, conv):
    cfg = synth.LayerConfig("t", K, N, bits, group, M, max(r, 1))
    L = synth.make_layer_torch(cfg, device="cuda", seed=31)
    f16 = conv == "f16"
    dtype, call = (torch.float16, b.modulora_f16_fwd) if f16 else (torch.bfloat16, b.modulora_fwd)
    if f16:
        bias = torch.randn(N, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).half()
        w = b.QWeightF16(L["qweight"], L["scales"], -2 * L["scales"], bias, K, N, bits, group)
        W = b.modulora_f16_dequant(w).double().t()
    else:
        w = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
        W = b.modulora_dequant(w).double().t()
    A, B = (L["A"] * 3, L["B"] * 30) if r else (None, None)
    X = torch.randn((M, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(2)).to(dtype)
    out = torch.full((M, N), float("nan"), dtype=dtype, device="cuda")
    b.modulora_profile_begin()
    Y, XA = call(w, X, A, B, 2.0, out)
    torch.cuda.synchronize()
    assert set(b.modulora_profile_end()) == {("f16_" if f16 else "") + "gemm_fwd_single"}
    X64 = X.double()
    ref, mag = X64 @ W, X64.abs() @ W.abs()
    if r:
        down = X64 @ A.double()
        assert bool(((XA.double() - down).abs() <= 2.0 ** -24 * (64 + K ** 0.5) * (X64.abs() @ A.double().abs())).all())
        ref, mag = ref + 2 * down @ B.double(), mag + 2 * (X64.abs() @ A.double().abs()) @ B.double().abs()
    if f16:
        ref = ref + bias.double()
    tol = (2.0 ** -11 if f16 else 2.0 ** -8) * ref.abs() + 2.0 ** -24 * (64 + K ** 0.5) * mag      # one rounding, fp32 sums
    assert bool(((Y.double() - ref).abs() <= tol).all()), float(((Y.double() - ref).abs() / tol).max())
    # a one-hot row picks a row of the weight, bit for bit
    hot = torch.zeros((M, K), dtype=dtype, device="cuda")
    hot[torch.arange(M), (torch.arange(M) * 37 + 5) % K] = 1.0
    picked = W[(torch.arange(M, device="cuda") * 37 + 5) % K].to(dtype)
    if f16:
        picked = (picked.float() + bias.float()).half()
    assert torch.equal(call(w, hot, None, None, 1.0)[0], picked)


@pytest.mark.parametrize("conv", ["bf16", "f16"])
@pytest.mark.parametrize("bits,K,N,M,r,group", [
    (4, 256, 256, 17, 8, 64),          # four units for eight waves
    (3, 384, 488, 252, 4, 32),         # groups of one block, the last unit of 40 n, a last row block of 28
    (2, 512, 264, 33, 9, 512),         # one group, the last unit of 8 n
    (4, 1024, 520, 100, 16, 128),      # nine units: a second round of one
    (3, 256, 1032, 40, 0, 64),         # no adapter
    (2, 768, 328, 64, 33, 96),
    (4, 640, 392, 98, 64, 128),
    (3, 6912, 264, 5, 1, 32),          # a handful of tokens that the backward streaming kernel does not take
])
def test_one_launch_backward(bits, K, N, M, r, group, conv):
    cfg = synth.LayerConfig("t", K, N, bits, group, M, max(r, 1))
    L = synth.make_layer_torch(cfg, device="cuda", seed=37)
    f16 = conv == "f16"
    dtype, call = (torch.float16, b.modulora_f16_bwd_input) if f16 else (torch.bfloat16, b.modulora_bwd_input)
    if f16:
        w = b.QWeightF16(L["qweight"], L["scales"], -2 * L["scales"], None, K, N, bits, group)
        W = b.modulora_f16_dequant(w).double()
    else:
        w = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
        W = b.modulora_dequant(w).double()
    A, B = (L["A"] * 30, L["B"] * 3) if r else (None, None)
    dY = torch.randn((M, N), device="cuda", generator=torch.Generator(device="cuda").manual_seed(2)).to(dtype)
    out = torch.full((M, K), float("nan"), dtype=dtype, device="cuda")
    b.modulora_profile_begin()
    dX, T = call(w, dY, A, B, 2.0, out)
    torch.cuda.synchronize()
    assert set(b.modulora_profile_end()) == {("f16_" if f16 else "") + "gemm_bwd_single"}
    dY64 = dY.double()
    ref, mag = dY64 @ W, dY64.abs() @ W.abs()
    if r:
        down = dY64 @ B.double().t()
        assert bool(((T.double() - down).abs() <= 2.0 ** -24 * (64 + N ** 0.5) * (dY64.abs() @ B.double().t().abs())).all())
        ref, mag = ref + 2 * down @ A.double().t(), mag + 2 * (dY64.abs() @ B.double().t().abs()) @ A.double().t().abs()
    tol = (2.0 ** -11 if f16 else 2.0 ** -8) * ref.abs() + 2.0 ** -24 * (64 + N ** 0.5) * mag      # one rounding, fp32 sums
    assert bool(((dX.double() - ref).abs() <= tol).all()), float(((dX.double() - ref).abs() / tol).max())
    # a one-hot row picks a row of the weight, bit for bit
    hot, at = torch.zeros((M, N), dtype=dtype, device="cuda"), (torch.arange(M, device="cuda") * 37 + 5) % N
    hot[torch.arange(M), at] = 1.0
    assert torch.equal(call(w, hot, None, None, 1.0)[0], W[at].to(dtype))
