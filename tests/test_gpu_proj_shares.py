"""Whole-K projections of up to 8 tokens on both sides of the lines that choose layout and shares (run with -m gpu)."""
import pytest
import torch

from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# panels per CU: up to 1/2, 1, 2 (with and without both places full), 3, 4, 6 and beyond; K: a wave's range of 1, 4, 6 and 7
# steps, one and two rings of 8, short of and at 3072, 6144, 8192 and 12288, ragged
@pytest.mark.parametrize("N", [2048, 4096, 5120, 8176, 12288, 16384, 20496, 32000])
@pytest.mark.parametrize("K", [200, 1016, 1536, 1800, 2048, 3072, 4104, 6136, 7168, 8192, 12296])
@pytest.mark.parametrize("M", [1, 4, 5, 8])
def test_projection_across_the_rules_lines(M, N, K):
    import paper_2408_11850_amd as amd
    gen = torch.Generator(device="cuda").manual_seed(N + K + M)
    w = torch.randn(N, K, generator=gen, device="cuda").mul_(0.05).to(torch.bfloat16)
    x = torch.randn(M, K, generator=gen, device="cuda").to(torch.bfloat16)
    ref = x.double() @ w.double().T
    d = amd.gemm(x, amd.binding.pack_matrices([w]), N).double() - ref
    # one rounding of 2^-24 per addition; no chain is longer than 60 additions, rows of y and columns of W are independent
    assert torch.isfinite(d).all()
    assert (d.norm() / ref.norm()).item() <= 2.0 ** -24 * 60 ** 0.5
    assert d.abs().max().item() <= 12 * 2.0 ** -24 * 60 ** 0.5 * ref.square().mean().sqrt().item()
