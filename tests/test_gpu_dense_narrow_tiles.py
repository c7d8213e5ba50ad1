"""The 128 x 96 tile of the prompt-time projection at its edges (run with -m gpu)."""
import pytest
import torch

import synth
from tests.test_gpu_dense_tiles import SMALL, test_dense_projection_of_every_tile as check_projection, tile
from tests.test_gpu_dense_wide_tiles import test_dense_and_chunked_prompt_passes_agree as check_prompt
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

NARROW = 3


# 256 tiles and 248, 240, 192 of them: whole tiles, one row more than a tile, N that ends two and four panels into a tile;
# K: 16 steps of 32, odd counts, longer than the ring many times over
@pytest.mark.parametrize("M,N,K", [(512, 6144, 512), (511, 6144, 2048), (385, 5920, 544), (500, 5888, 608), (129, 9152, 2144), (1023, 3072, 512)])
@pytest.mark.parametrize("epilogue", [0, 1, 2])      # 0 and 1, fp32 results, take 128 x 128 (test_prompt_tiles.py)
def test_projection(M, N, K, epilogue):
    assert tile(M, N, K - 32 * (K // 32 - 15)) == SMALL          # 15 steps
    check_projection(M, N, K, NARROW, epilogue)


# QKV with its rotation and page append: a tile holds three quarters of a head of 128, one and a half of 64
@pytest.mark.parametrize("shape", [synth.ModelShape(2, 512, 32, 8, 256, 1024, 128), synth.ModelShape(2, 512, 64, 16, 256, 1024, 64)])
def test_dense_and_chunked_prompt_passes(shape):
    check_prompt(shape, 512, NARROW)
