"""When spec_gemm writes to its workspace (host only)."""
import pytest

import paper_2408_11850_amd as amd


@pytest.mark.parametrize("M,N,K,uses", [(1, 2048, 2048, 0), (8, 8192, 28672, 0), (17, 38400, 7168, 0), (1, 256, 2048, 1), (32, 4096, 11008, 1)])
def test_workspace_use_follows_kernel_and_alignment(M, N, K, uses):
    lib = amd.load_library()
    assert lib.spec_gemm_uses_work(0x1000, 0x2000, M, N, K) == uses
    assert lib.spec_gemm_uses_work(0x1002, 0x2000, M, N, K) == 1      # K slices take any address of an element
    assert lib.spec_gemm_uses_work(0x1000, 0x2008, M, N, K) == 1


def test_refused_shapes():
    lib = amd.load_library()
    for M, N, K in ((0, 64, 64), (33, 64, 64), (1, 40, 64), (1, 64, 60)):
        assert lib.spec_gemm_uses_work(0x1000, 0x2000, M, N, K) == amd.SPEC_E_INVAL
