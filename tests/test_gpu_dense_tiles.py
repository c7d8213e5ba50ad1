"""The prompt-time projection with both tile sizes, at the edges of tiles, rounds and the operand ring (run with -m gpu)."""
import pytest
import torch

from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# K: 1, 2, 3, 5, 8 and 67 steps of 32 (shorter than the ring, odd counts); M and N one beside a tile; 1023 x 22016 and
# 511 x 24576 take the large tile, the rest the small one
@pytest.mark.parametrize("M,N,K", [(1, 32, 32), (65, 96, 64), (127, 128, 96), (128, 160, 160), (129, 2080, 256),
                                   (257, 512, 2144), (511, 6144, 96), (1023, 4128, 64), (1023, 22016, 96), (511, 24576, 64)])
@pytest.mark.parametrize("epilogue", [0, 1, 2])
def test_dense_projection_of_every_tile(M, N, K, epilogue):
    import paper_2408_11850_amd as amd
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    w, x = rnd(N, K).mul_(0.05).to(torch.bfloat16), rnd(M, K).to(torch.bfloat16)
    ref = x.double() @ w.double().T
    packed = amd.binding.pack_matrices([w])
    # fp32: a chain of K / 32 additions, rounding errors independent, 12 deviations for the largest of 2^24 elements; the
    # products of silu(g) * u carry those of g and u, each about as large as its factor
    f32 = 2.0 ** -24 * (K / 32 + 8) ** 0.5 * 2
    if epilogue == 2:
        got = amd.dense_gemm(x, packed, N, 2).double()
        ref = ref.view(M, -1, 2, 16)
        scale = (ref[:, :, 0].square().mean().sqrt() * (1 + ref[:, :, 1].abs().max())).item() * 2
        ref = (torch.nn.functional.silu(ref[:, :, 0]) * ref[:, :, 1]).reshape(M, -1)
        rel = 2.0 ** -8          # an element's own rounding to bf16: 8 significant bits, at worst half a unit of 2^-7 above a power of two
    else:
        y0 = rnd(M, N)
        got = amd.dense_gemm(x, packed, N, epilogue, y0.clone() if epilogue else None).double()
        ref = ref + y0.double() if epilogue else ref
        scale, rel = ref.square().mean().sqrt().item(), 0.0
    assert got.shape == ref.shape and torch.isfinite(got).all()
    assert ((got - ref).abs() - rel * ref.abs()).max().item() <= 12 * f32 * scale
    assert ((got - ref).norm() / ref.norm()).item() <= rel + f32
