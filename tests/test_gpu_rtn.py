"""GPU parity of the round-to-nearest quantizer + packer (C ABI) against the numpy oracle:
bit-exact words, scales and zero points; and the round trip through the library's own
dequantizer within the error bound."""
import numpy as np
import pytest
import torch

import oracle
from oracle import rtn
from paper_2309_16119_amd import binding as b

pytestmark = pytest.mark.gpu


def weight(N, K, seed):
    """Weights like a trained linear layer's: normal, with a heavy-tailed per-row scale and a few
    outliers; plus degenerate rows (all zero, all positive, all negative, constant)."""
    rng = np.random.default_rng(seed)
    W = (rng.normal(size=(N, K)) * rng.lognormal(sigma=1.0, size=(N, 1)) * 0.02).astype(np.float32)
    out = rng.integers(0, N * K, size=max(1, N * K // 500))
    W.reshape(-1)[out] *= 8
    W[0] = 0.0
    W[1] = np.abs(W[1])
    W[2] = -np.abs(W[2])
    W[3] = 0.37
    W[4, : K // 2] = 0.0
    return W


@pytest.mark.parametrize("bits,K,N,group", [
    (4, 256, 256, 64), (3, 416, 296, 32), (2, 448, 8, 64), (4, 32, 1032, 32), (3, 1024, 520, 1024),
    (2, 2048, 264, 128), (3, 2240, 72, 160), (4, 3072, 136, 1536), (2, 4096, 64, 4096), (3, 4096, 4096, 128),
])
def test_quantize_bit_exact(bits, K, N, group):
    W = weight(N, K, seed=bits * 1000 + group)
    qw = b.modulora_quantize_rtn(torch.from_numpy(W).cuda(), bits, group)
    q_ref, s_ref, z_ref = rtn.quantize_packed(W, bits, group)
    assert np.array_equal(qw.scales.cpu().numpy().view(np.uint16), s_ref)
    assert np.array_equal(qw.zeros.cpu().numpy(), z_ref)
    assert np.array_equal(qw.qweight.cpu().numpy().view(np.uint32), q_ref)


def test_quantize_then_dequantize_full_size_within_the_bound():
    """LLaMA-65B up projection (8192 -> 22016), 3-bit, group 128: quantize on the GPU, materialize
    with the library's dequantizer, check |w - what| <= scale (1/2 + 2^-20) + the bfloat16 rounding
    of what (2^-9 relative) everywhere, on the GPU; sampled columns bit-exact against the oracle."""
    K, N, bits, group = 8192, 22016, 3, 128
    g = torch.Generator(device="cuda").manual_seed(11)
    W = torch.randn((N, K), device="cuda", generator=g) * 0.02
    qw = b.modulora_quantize_rtn(W, bits, group)
    What = b.modulora_dequant(qw).float()                                   # [N][K]
    s = qw.scales.float().t().repeat_interleave(group, dim=1)              # [N][K]
    bound = s * (0.5 + 2.0 ** -20) + What.abs() * 2.0 ** -8
    assert bool(torch.all((W - What).abs() <= bound))
    cols = [0, 1, 4097, 22015]
    Wc = W[cols].cpu().numpy()
    q_ref, s_ref, z_ref = rtn.quantize_packed(Wc, bits, group)
    assert np.array_equal(qw.qweight[:, cols].cpu().numpy().view(np.uint32), q_ref)
    assert np.array_equal(qw.scales[:, cols].cpu().numpy().view(np.uint16), s_ref)
    assert np.array_equal(qw.zeros[:, cols].cpu().numpy(), z_ref)


def test_quantized_layer_runs_through_the_forward_pass():
    """The quantizer's output is a valid layer: forward of the library against the oracle's
    forward on the same (GPU-independent) oracle-quantized weight."""
    from paper_2309_16119_amd import synth
    from gpu_util import assert_bar, f64
    K, N, M, bits, group = 512, 384, 40, 4, 128
    W = weight(N, K, seed=3)
    q_ref, s_ref, z_ref = rtn.quantize_packed(W, bits, group)
    qw = b.modulora_quantize_rtn(torch.from_numpy(W).cuda(), bits, group)
    rng = np.random.default_rng(4)
    X = synth.f32_to_bf16_bits(rng.normal(size=(M, K)).astype(np.float32))
    Xd = torch.from_numpy(X.view(np.int16)).cuda().view(torch.bfloat16)
    Y, _ = b.modulora_fwd(qw, Xd, None, None, 0.0)
    Yr, _ = oracle.fwd(q_ref, s_ref, z_ref, K, N, bits, group, X, None, None, 0.0)
    assert_bar("Y", f64(Y), Yr)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("K,N,group", [(32, 8, 32), (160, 72, 32), (192, 64, 64), (384, 136, 128), (256, 8, 256),
                                       (768, 200, 256)])
def test_one_pass_kernel_at_tile_edges_and_ties(bits, K, N, group):
    """The one-pass kernel (groups of 32 .. 256) where its 64-row and 128- / 256-input tiles end
    inside the matrix, on weights that make its shortcut around the division decide: quotients
    that are exact half-integers, and their float32 neighbours on either side."""
    rng = np.random.default_rng(100 * bits + K)
    W = weight(N, K, seed=bits + K)
    maxq = (1 << bits) - 1
    half = rng.integers(0, 2 * maxq + 1, size=(N, K)).astype(np.float32) / 2 - maxq // 2
    half.reshape(N, K // group, group)[:, :, :2] = [-(maxq // 2), maxq - maxq // 2]     # the whole range: scale = 2^-5
    ties = (half * np.float32(2.0 ** -5)).astype(np.float32)
    nudge = rng.integers(-1, 2, size=(N, K))
    ties = np.where(nudge < 0, np.nextafter(ties, np.float32(-9)), np.where(nudge > 0, np.nextafter(ties, np.float32(9)), ties))
    ties.reshape(N, K // group, group)[:, :, :2] = np.float32(2.0 ** -5) * np.array([-(maxq // 2), maxq - maxq // 2], np.float32)
    W[N // 2:] = ties[N // 2:]
    qw = b.modulora_quantize_rtn(torch.from_numpy(W).cuda(), bits, group)
    q_ref, s_ref, z_ref = rtn.quantize_packed(W, bits, group)
    assert np.array_equal(qw.scales.cpu().numpy().view(np.uint16), s_ref)
    assert np.array_equal(qw.zeros.cpu().numpy(), z_ref)
    assert np.array_equal(qw.qweight.cpu().numpy().view(np.uint32), q_ref)


@pytest.mark.parametrize("d_out,d_in,bits,group,status", [
    (64, 256, 5, 64, 3), (64, 256, 0, 64, 3), (64, 256, 4, 0, 4), (64, 256, 4, -32, 4), (64, 256, 4, 48, 4), (64, 256, 4, 512, 4),
    (64, 250, 4, 32, 2), (12, 256, 4, 64, 2), (0, 256, 4, 64, 2), (64, 0, 4, 64, 2),
])
def test_refused_shapes(monkeypatch, d_out, d_in, bits, group, status):
    """The library's own status, without a size query ahead of the call."""
    class Library:
        modulora_quantize_rtn, modulora_status_string = b.lib.modulora_quantize_rtn, b.lib.modulora_status_string
    monkeypatch.setattr(b, "lib", Library)
    with pytest.raises(b.ModuloraError) as e:
        b.modulora_quantize_rtn(torch.zeros((d_out, d_in), device="cuda"), bits, group)
    assert e.value.status == status
    b.modulora_quantize_rtn(torch.zeros((64, 256), device="cuda"), 4, 64)
