"""Sizes at which the estimates choose what no other test reaches: 128-row tiles for many row blocks, sliced and
whole rounds of them, the sliced contractions that project by themselves, and the kernel for up to 1024 tokens
for a small layer whose output is whole 16-column tiles but no whole column blocks.  Against the product with the
dequantized weight in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2309_16119_amd import binding as b, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("conv,direction,bits,K,N,M,r,group,kernel", [
    ("bf16", "fwd", 4, 5376, 640, 1535, 0, 128, "gemm_fwd_128x256"),         # twelve row blocks, the last one row short, sliced
    ("bf16", "bwd", 3, 256, 4864, 1716, 0, 64, "gemm_bwd_128x256"),          # one column block, 52 rows in the last block
    ("f16", "fwd", 4, 768, 18304, 794, 0, 128, "f16_gemm_fwd"),              # more than 256 whole tiles, no adapter
    ("f16", "fwd", 3, 11648, 256, 1061, 0, 128, "f16_gemm_fwd"),             # 37 rows in the last block
    ("bf16", "fwd", 4, 2560, 1040, 40, 16, 32, "gemm_fwd_direct"),           # 16 columns in the last block
    ("f16", "fwd", 3, 6912, 608, 25, 4, 64, "f16_gemm_fwd_direct"),
    ("bf16", "fwd", 2, 3328, 912, 458, 8, 128, "gemm_fwd_direct"),
    # sliced contractions with the projection as a side job: in idle units
    ("bf16", "fwd", 2, 6656, 6656, 1024, 8, 64, "sliced"),
    ("bf16", "bwd", 2, 6656, 6656, 1024, 8, 64, "sliced"),
    ("f16", "fwd", 4, 2336, 272, 1100, 16, 32, "sliced"),                    # the contraction ends inside a step of 64; 16 columns over
    ("bf16", "bwd", 3, 256, 2056, 1300, 33, 128, "sliced"),                  # ... and inside one of 32; rank no multiple of four
    ("f16", "bwd", 4, 384, 3840, 118, 32, 128, "sliced"),                    # one row block
    ("bf16", "fwd", 4, 5376, 640, 1535, 1, 128, "sliced"),
    # ... and ahead of every workgroup's share of the product
    ("bf16", "fwd", 4, 4736, 512, 1475, 8, 128, "sliced"),
    ("f16", "fwd", 2, 8064, 2432, 1072, 16, 128, "sliced"),
    ("bf16", "bwd", 2, 2560, 3712, 1449, 8, 128, "sliced"),
])
def test_chosen_by_the_estimates(conv, direction, bits, K, N, M, r, group, kernel):
    cfg = synth.LayerConfig("t", K, N, bits, group, M, r)
    L = synth.make_layer_torch(cfg, device="cuda", seed=19)
    f16 = conv == "f16"
    dtype = torch.float16 if f16 else torch.bfloat16
    if f16:
        w = b.QWeightF16(L["qweight"], L["scales"], -2 * L["scales"], None, K, N, bits, group)
        What, calls = b.modulora_f16_dequant(w), (b.modulora_f16_fwd, b.modulora_f16_bwd_input)
    else:
        w = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, bits, group)
        What, calls = b.modulora_dequant(w), (b.modulora_fwd, b.modulora_bwd_input)
    A, B = (L["A"], L["B"]) if r else (None, None)
    fwd = direction == "fwd"
    act = (L["X"] if fwd else L["dY"]).to(dtype)
    out = torch.full((M, N if fwd else K), float("nan"), dtype=dtype, device="cuda")
    b.modulora_profile_begin()
    got, P = calls[0 if fwd else 1](w, act, A, B, 2.0, out)
    torch.cuda.synchronize()
    names = set(b.modulora_profile_end())
    if kernel == "sliced":      # the product and its second launch, nothing ahead of them
        big = {"f16_gemm_" + direction} if f16 else {"gemm_%s_%dx256" % (direction, rows) for rows in (128, 256)}
        assert len(names) == 2 and len(names & big) == 1 and len(names & {n + "_fixup" for n in big}) == 1, names
    else:
        assert kernel in names, names
    a64, W = act.double(), What.double().t() if fwd else What.double()      # What [N][K]
    ref, mag = a64 @ W, a64.abs() @ W.abs()
    if r:
        down, up = (A.double(), B.double()) if fwd else (B.double().t(), A.double().t())
        Pr = a64 @ down
        # fp32 sums of exact products, of as many terms as the contraction has
        assert bool(((P.double() - Pr).abs() <= 2.0 ** -24 * (64 + len(down) ** 0.5) * (a64.abs() @ down.abs())).all())
        ref, mag = ref + 2 * Pr @ up, mag + 2 * (a64.abs() @ down.abs()) @ up.abs()
    # one rounding of the output and the fp32 accumulation
    tol = (2.0 ** -11 if f16 else 2.0 ** -8) * ref.abs() + 2.0 ** -24 * (64 + (K if fwd else N) ** 0.5) * mag
    assert bool(((got.double() - ref).abs() <= tol).all()), float(((got.double() - ref).abs() / tol).max())
