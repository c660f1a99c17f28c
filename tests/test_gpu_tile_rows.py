"""The large-tile kernel's instantiation with 192 rows, where the estimates choose it: nine rows and one row in the last block,
a last column block of 136 and of 32, a contraction that ends inside a step of 64, more than one round of tiles, no adapter
and ranks of one and two extension steps.  Against the product with the dequantized weight in 64 bits."""
import pytest
import torch

from test_gpu_tile_choice import test_chosen_by_the_estimates as check_product

from paper_2309_16119_amd import binding as b, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("conv", ["bf16", "f16"])
@pytest.mark.parametrize("direction,bits,K,N,M,r,group", [
    ("fwd", 4, 544, 2440, 3465, 8, 32),
    ("bwd", 4, 2464, 552, 3465, 16, 32),
    ("fwd", 3, 768, 2560, 3457, 0, 128),
    ("bwd", 3, 2560, 776, 3457, 32, 128),
    ("fwd", 2, 1664, 11008, 1546, 8, 128),
    ("bwd", 2, 11008, 1664, 1546, 3, 64),
])
def test_rows_of_192(conv, direction, bits, K, N, M, r, group):
    name = ("f16_gemm_%s" if conv == "f16" else "gemm_%s_192x256") % direction
    check_product(conv, direction, bits, K, N, M, r, group, name)


def test_rows_of_192_reproduce_the_weight_bit_exactly():
    """One-hot activations: every output is a single weight, with the bit pattern of the materialized one."""
    K, N, M = 768, 2560, 3457
    L = synth.make_layer_torch(synth.LayerConfig("t", K, N, 3, 128, 1, 1), device="cuda", seed=3)
    w = b.QWeight(L["qweight"], L["scales"], L["zeros"], K, N, 3, 128)
    hot = torch.arange(M, device="cuda") * 5 % K
    rows = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda")
    rows[torch.arange(M, device="cuda"), hot] = 1.0
    b.modulora_profile_begin()
    Y, _ = b.modulora_fwd(w, rows, None, None, 1.0)
    torch.cuda.synchronize()
    assert set(b.modulora_profile_end()) == {"gemm_fwd_192x256"}
    assert torch.equal(Y.view(torch.int16), b.modulora_dequant(w).t()[hot].contiguous().view(torch.int16))
