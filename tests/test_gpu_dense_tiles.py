"""The prompt-time projection with every tile, at the edges of tiles, rounds and the operand ring (run with -m gpu)."""
import ctypes as C

import pytest
import torch

from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


LARGE, SMALL, WIDE = 0, 1, 2      # 256 x 256, 128 x 128, 256 x 192


def tile(M, N, K):
    """The tile that the library takes for these sizes."""
    import paper_2408_11850_amd as amd
    amd.load_library()
    f = C.CDLL(amd.LIB_PATH)._Z10dense_tileiii
    f.argtypes = [C.c_int] * 3
    return f(M, N // 16, K // 32)


# K: 1, 2, 3, 5, 7, 8, 10 and 67 steps of 32 (shorter than the rings, odd counts); M and N one beside a tile.  In the large
# tile's rows an XCD has 13, 14, 15, 8, 11 and 5 tile columns, i.e. groups of 4 and a last one of 1, 2, 3, 4, 3 and 1; the last
# XCD is short of columns in all but the last row; the last two take two rounds of tiles
@pytest.mark.parametrize("M,N,K,which", [(1, 32, 32, SMALL), (65, 96, 64, SMALL), (127, 128, 96, SMALL), (128, 160, 160, SMALL),
                                         (129, 2080, 256, SMALL), (257, 512, 2144, SMALL), (511, 6144, 96, SMALL),
                                         (1023, 4128, 64, WIDE), (1023, 22016, 96, WIDE), (511, 24576, 64, WIDE),
                                         (509, 25312, 32, LARGE), (509, 25312, 96, LARGE), (509, 27904, 64, LARGE),
                                         (511, 29632, 160, LARGE), (1021, 15584, 96, LARGE), (1300, 21216, 320, LARGE),
                                         (3001, 10208, 224, LARGE)])
@pytest.mark.parametrize("epilogue", [0, 1, 2])
def test_dense_projection_of_every_tile(M, N, K, which, epilogue):
    import paper_2408_11850_amd as amd
    assert tile(M, N, K) == which
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
