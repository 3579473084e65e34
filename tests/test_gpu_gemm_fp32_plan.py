"""fp32 GEMM: every tile height and K split that the time model may choose gives the reference kernel's bits (0 differing
bits: the summation order does not depend on them), at batch sizes around the edges of 32- and 128-row tiles, of groups of
eight row tiles and of rounds of 256 work items, also when the caller's workspace holds only a smaller split's planes."""
import pytest
import torch

from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N,leaf,kf", [(1536, 2048, 32, 3), (4096, 132, 128, 1)])
@pytest.mark.parametrize("M", [1, 32, 33, 65, 128, 129, 300, 450, 600, 1025, 1200])
def test_plan_bits(K, N, leaf, kf, M):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(M)
    X = torch.randn((M, K), generator=g, device="cuda:0")
    W = torch.randn((K, N), generator=g, device="cuda:0") * 0.02
    want = tb.tbik_gemm_reference_f32(X, W, leaf, kf)[1].view(torch.int32)
    assert torch.equal(tb.tbik_gemm_f32(X, W, leaf, kf).view(torch.int32), want)
    need = tb.gemm_workspace_bytes(M, N, K, leaf, kf)
    ws = torch.full((max(need, 256) // 4,), float("nan"), dtype=torch.float32, device="cuda:0")
    assert torch.equal(tb.tbik_gemm_f32(X, W, leaf, kf, workspace=ws).view(torch.int32), want)
    for variant in (2, 3):                                        # 128- and 32-row tiles
        tb.tbik_set_gemm_variant(variant)
        assert torch.equal(tb.tbik_gemm_f32(X, W, leaf, kf).view(torch.int32), want), variant
        for P in (2, 8):
            parts = tb.tbik_gemm_shard_partials_f32(X, W, leaf, kf, P)
            assert torch.equal(tb.tbik_tree_combine(parts, out_dtype=torch.float32).view(torch.int32), want), (variant, P)
    tb.tbik_set_gemm_variant(0)


@pytest.mark.parametrize("M,N,K,leaf,rule,plan", [(1200, 2048, 1536, 96, 1, 2), (321, 4096, 2048, 256, 1, 2), (129, 4096, 4096, 256, 4, 8)])
def test_smaller_workspace_takes_a_smaller_split(M, N, K, leaf, rule, plan):
    """The model's split takes more planes than the older rule's: a workspace of the rule's planes is enough, the bits are the same,
    and less is refused."""
    X, W = torch.randn((M, K), device="cuda:0"), torch.randn((K, N), device="cuda:0")
    want = tb.tbik_gemm_reference_f32(X, W, leaf, 1)[1]
    assert tb.gemm_f32_workspace_bytes(M, N, K, leaf, 1) == plan * M * N * 4
    for planes in (0 if rule == 1 else rule, plan - 1, plan):
        ws = torch.full((planes * M * N,), float("nan"), dtype=torch.float32, device="cuda:0")
        assert torch.equal(tb.tbik_gemm_f32(X, W, leaf, 1, workspace=ws).view(torch.int32), want.view(torch.int32)), planes
    if rule > 1:
        with pytest.raises(tb.TbikError):
            tb.tbik_gemm_f32(X, W, leaf, 1, workspace=torch.empty(rule * M * N - 64, dtype=torch.float32, device="cuda:0"))
