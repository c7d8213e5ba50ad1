"""Whole-K projections of up to 8 tokens on both sides of the lines that choose layout and shares (run with -m gpu)."""
import pytest
import torch

from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# panels per CU: up to 1/2, 1, 2 (with and without both places full), 3, 4, 6 and beyond; K: a wave's range of 1, 2, 3, 4, 5,
# 6, 7 and 8 steps, one and two rings of 8, both sides of 3072, 6144, 8192 and 12288, ragged
@pytest.mark.parametrize("N", [2048, 4096, 5120, 8176, 12288, 16384, 20496, 32000])
@pytest.mark.parametrize("K", [200, 512, 768, 1016, 1280, 1536, 1768, 1800, 2048, 3064, 3072, 4104, 6136, 6144, 7168, 8192, 8200,
                               12280, 12288, 12296])
def test_projection_across_the_rules_lines(N, K):
    import paper_2408_11850_amd as amd
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    w = torch.randn(N, K, generator=gen, device="cuda").mul_(0.05).to(torch.bfloat16)
    packed = amd.binding.pack_matrices([w])
    x8 = torch.randn(8, K, generator=gen, device="cuda").to(torch.bfloat16)
    exact = x8.double() @ w.double().T
    for M in (1, 4, 5, 8):
        x, ref = x8[:M], exact[:M]
        d = amd.gemm(x, packed, N).double() - ref
        # one rounding of 2^-24 per addition; no chain is longer than 60 additions, rows of y and columns of W are independent
        assert torch.isfinite(d).all(), M
        assert (d.norm() / ref.norm()).item() <= 2.0 ** -24 * 60 ** 0.5, M
        assert d.abs().max().item() <= 12 * 2.0 ** -24 * 60 ** 0.5 * ref.square().mean().sqrt().item(), M
