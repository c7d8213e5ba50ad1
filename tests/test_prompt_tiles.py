"""Which results the 128 x 96 tile of the prompt-time projection is taken for (host only)."""
import ctypes as C

import pytest

import paper_2408_11850_amd as amd

SMALL, NARROW = 1, 3
STORE, RESID, SWIGLU, ROPE128, ROPE64 = range(5)


# 256, 240, 224 and 192 tiles of 128 x 96
@pytest.mark.parametrize("M,N,K", [(511, 6144, 2048), (511, 5760, 2048), (1023, 2688, 4096), (511, 4608, 4096), (129, 9152, 512)])
def test_fp32_results_keep_128_x_128(M, N, K):
    amd.load_library()
    f = C.CDLL(amd.LIB_PATH)._Z14dense_epi_tileiiii
    f.argtypes = [C.c_int] * 4
    of = [f(M, N // 16, K // 32, epi) for epi in (STORE, RESID, SWIGLU, ROPE128, ROPE64)]
    assert of == [SMALL, SMALL, NARROW, NARROW, NARROW]
    assert [f(M, N // 16, 15, epi) for epi in range(5)] == [SMALL] * 5


def test_other_tiles_do_not_depend_on_the_results():
    amd.load_library()
    lib = C.CDLL(amd.LIB_PATH)
    shape, of = lib._Z10dense_tileiii, lib._Z14dense_epi_tileiiii
    shape.argtypes, of.argtypes = [C.c_int] * 3, [C.c_int] * 4
    seen = set()
    for M in (1, 100, 255, 511, 1023, 2047, 4095):
        for N in (512, 3072, 6144, 8192, 12288, 22016, 57344):
            for K in (256, 2048, 4096, 11008):
                t = shape(M, N // 16, K // 32)
                seen.add(t)
                assert t == NARROW or all(of(M, N // 16, K // 32, epi) == t for epi in range(5)), (M, N, K)
    assert seen == {0, 1, 2, 3}
