"""fp32 GEMM on 32-row tiles: the reference kernel's bits where the work items are one short of, as many as and one more than a
multiple of the 512 workgroups that share them, at K-loops shorter than, as long as and longer than the ring of LDS stages."""
import pytest
import torch

from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,leaf", [(32, 32), (96, 96), (64, 32), (128, 32), (512, 32)])
@pytest.mark.parametrize("M,N,items", [(2330, 896, 511), (1024, 2048, 512), (608, 3456, 513), (2048, 2044, 1024), (1300, 3200, 1025)])
def test_items(M, N, items, K, leaf):
    assert ((M + 31) // 32) * ((N + 127) // 128) == items
    g = torch.Generator(device="cuda:0")
    g.manual_seed(M + K)
    X = torch.randn((M, K), generator=g, device="cuda:0")
    W = torch.randn((K, N), generator=g, device="cuda:0")
    want = tb.tbik_gemm_reference_f32(X, W, leaf, 1)[0]
    tb.tbik_set_gemm_variant(tb.VARIANT_T32)
    try:
        got = tb.tbik_gemm_shard_partials_f32(X, W, leaf, 1, 1)
    finally:
        tb.tbik_set_gemm_variant(tb.VARIANT_AUTO)
    assert torch.equal(got.reshape(M, N).view(torch.int32), want.reshape(M, N).view(torch.int32))
