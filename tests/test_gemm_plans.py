"""The plans that GEMM calls follow, seen on the host (no device is needed): which batches are cut into two pieces, by the planes
that a call asks for."""
import os

import pytest


@pytest.fixture(scope="module")
def L():
    from paper_2511_17826_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2511_17826_amd import build
        build.build()
    return binding.lib()


def planes(n, M, N):
    return n * M * N * 4


@pytest.mark.parametrize("M,N,K,rest", [(1095, 4096, 4096, 71), (1100, 4096, 4096, 76), (690, 6144, 4096, 50), (838, 5120, 4096, 70)])
def test_plain_8_bit_batches_are_cut(L, M, N, K, rest):
    """Whole, these take two rounds of 128-row tiles and no planes; cut, the last rows are split in two."""
    assert L.tbik_gemm_fp8_workspace_bytes(M, N, K, 256, 1) == planes(2, rest, N)


@pytest.mark.parametrize("M,N", [(674, 6144), (808, 5120)])
def test_mxfp8_batches_are_cut(L, M, N):
    scales = (-(-M // 128) * 128 + N) * 4096 // 32
    assert L.tbik_gemm_mxfp8_workspace_bytes(M, N, 4096, 256, 1) == planes(4, M - 128 * (256 // (N // 128)), N) + scales


def test_batches_that_a_cut_does_not_pay_for_stay_whole(L):
    assert L.tbik_gemm_fp8_workspace_bytes(1064, 4096, 3072, 768, 1) == 0
