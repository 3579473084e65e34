"""The plans that GEMM calls follow, seen on the host (no device is needed): which batches are cut into two pieces, by the planes
that a call asks for, and which kernel, tile and split each piece gets."""
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


def route(*shape):
    from paper_2511_17826_amd import binding
    return binding.gemm_route(*shape)


def test_routes(L):
    assert route("bf16", 77, 4096, 12288, 256, 3) == [(77, "tiles", 96, 8)]
    assert route("bf16", 97, 4096, 12288, 256, 3) == [(97, "tiles", 128, 8)]
    assert route("fp16", 1100, 4096, 4096, 256, 1) == [(1024, "tiles", 128, 1), (76, "tiles", 64, 4)]
    assert route("bf16", 5, 12, 256, 256, 1) == [(5, "reference", 0, 0)]
    assert route("f32", 600, 2048, 6144, 128, 3) == [(600, "tiles", 32, 4)]
    assert route("fp8", 16, 4096, 12288, 256, 3) == [(16, "slices", 0, 0)]
    assert route("fp8", 33, 4096, 4096, 256, 1) == [(33, "tiles", 32, 4)]
    assert route("fp8", 16, 4096, 4096, 64, 1) == [(16, "reference", 0, 0)]          # superleaves shorter than a stage
    assert route("mxfp6", 4097, 1024, 2048, 256, 1) == [(4096, "tiles", 128, 1), (1, "slices", 0, 0)]
    assert route("mxfp4", 0, 1024, 2048, 256, 1) == []


def test_a_forced_variant_is_what_the_route_tells(L):
    from paper_2511_17826_amd import binding as tb
    try:
        tb.tbik_set_gemm_variant(tb.VARIANT_T64)
        assert route("fp8", 16, 4096, 4096, 256, 1)[0][1:3] == ("tiles", 64) and route("bf16", 77, 4096, 12288, 256, 3)[0][2] == 64
        tb.tbik_set_gemm_variant(tb.VARIANT_REFERENCE)
        assert route("mxfp4", 16, 4096, 4096, 256, 1)[0][1] == "reference"
    finally:
        tb.tbik_set_gemm_variant(tb.VARIANT_AUTO)


def test_route_arguments(L):
    import ctypes as C
    r = (C.c_int * 8)()
    assert L.tbik_gemm_route(1, 0, 4, 256, 500, 64, 1, r) == 2 and L.tbik_gemm_route(9, 0, 4, 256, 512, 64, 1, r) == 4
    assert L.tbik_gemm_route(1, 0, 4, 256, 512, 64, 1, None) == 1 and L.tbik_gemm_route(3, 0, 4, 256, 512, 32, 1, r) == 2


@pytest.mark.parametrize("kind,M,N,K,leaf,k_first,kernel", [
    # (M, N, K and trees of the layers that the benchmark runs)
    ("fp8", 1, 4096, 4096, 256, 1, "slices"), ("fp8", 32, 4096, 12288, 256, 3, "slices"), ("fp8", 32, 6144, 4096, 256, 1, "slices"),
    ("mxfp8", 16, 4096, 12288, 256, 3, "slices"), ("mxfp6", 32, 4096, 12288, 256, 3, "slices"), ("mxfp4", 32, 4096, 12288, 256, 3, "slices"),
    # long K on few channels: the tiled kernels spread it over more compute units (8-bit 15.1 us as slices, 11.1 as tiles)
    ("fp8", 32, 1024, 16384, 256, 4, "tiles"), ("fp8", 32, 256, 12288, 256, 3, "tiles"), ("fp8", 16, 256, 24576, 512, 3, "tiles"),
    ("mxfp8", 16, 1024, 16384, 256, 4, "tiles"), ("mxfp6", 32, 1024, 16384, 256, 4, "tiles"), ("mxfp4", 32, 1024, 24576, 512, 3, "tiles"),
    ("mxfp4", 16, 1024, 16384, 256, 4, "slices"), ("fp8", 16, 4096, 16384, 256, 4, "slices"),
    # more slices than compute units and long K: 28.6 us as slices, 20.9 as tiles
    ("fp8", 32, 6144, 12288, 256, 3, "tiles"), ("mxfp4", 32, 6144, 12288, 256, 3, "tiles"),
    # one and two superleaves: one and two of a workgroup's wavefronts work
    ("fp8", 16, 4096, 4096, 4096, 1, "slices"), ("fp8", 16, 12288, 4096, 4096, 1, "tiles"), ("mxfp8", 1, 12288, 4096, 2048, 1, "tiles"),
    ("mxfp8", 1, 6144, 4096, 2048, 1, "slices"), ("mxfp4", 32, 8192, 4096, 4096, 1, "slices"), ("mxfp6", 16, 12288, 4096, 4096, 1, "slices"),
    ("fp8", 16, 8192, 2048, 2048, 1, "slices"), ("mxfp6", 16, 12288, 512, 512, 1, "tiles")])
def test_slices_where_they_are_quicker(L, kind, M, N, K, leaf, k_first, kernel):
    assert route(kind, M, N, K, leaf, k_first)[0][1] == kernel


@pytest.mark.parametrize("M,N,K,leaf,k_first", [(77, 2048, 6144, 128, 3), (1100, 2048, 6144, 128, 3), (600, 4096, 4096, 128, 1), (1100, 4096, 4096, 256, 1)])
def test_fp32_batches_on_two_workgroups_per_compute_unit(L, M, N, K, leaf, k_first):
    """A ragged last round of 32-row tiles costs what a model of 512 workgroups says, and these batches take them: 4 to 13 % less time."""
    assert route("f32", M, N, K, leaf, k_first)[0][2] == 32


def test_fp32_splits_no_further_than_they_pay(L):
    """30 row and column tiles split in eight leave each item a compute unit (19.2 us); in sixteen, the combine eats the gain (21.1)."""
    assert route("f32", 88, 1280, 4096, 256, 1) == [(88, "tiles", 32, 8)]
