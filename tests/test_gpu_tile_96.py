"""GPU tests of the 96-row tile that 16-bit batches of 65..96 rows take: every bit equal to the reference kernel's and nothing
written past the last row, at both ends of the range and beside it, for whole and ragged columns, both operand formats, 16-bit,
fp32 and shard-partial outputs."""
import pytest
import torch

from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N,leaf,k_first", [(4096, 6144, 256, 1), (4096, 6136, 256, 1), (5120, 7168, 128, 5), (12288, 4096, 256, 3)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_bits(dtype, K, N, leaf, k_first):
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    f16 = dtype == torch.float16
    gemm, ref = (tb.tbik_gemm_f16, tb.tbik_gemm_reference_f16) if f16 else (tb.tbik_gemm, tb.tbik_gemm_reference)
    partials = tb.tbik_gemm_shard_partials_f16 if f16 else tb.tbik_gemm_shard_partials
    W = torch.randn((K, N), generator=g, device="cuda").mul_(0.05).to(dtype)
    X = torch.randn((97, K), generator=g, device="cuda").to(dtype)
    want = ref(X, W, leaf, k_first, 1, out_dtype=torch.float32)[1]
    for M in (64, 65, 79, 95, 96, 97):
        assert (tb.gemm_route("fp16" if f16 else "bf16", M, N, K, leaf, k_first)[0][2] == 96) == (65 <= M <= 96), M
        for out_dtype in (dtype, torch.float32):
            t = torch.full((M + 2, N), -7.0, dtype=out_dtype, device="cuda")
            gemm(X[:M], W, leaf, k_first, out=t[1:M + 1])
            assert torch.equal(t[1:M + 1], want[:M].to(out_dtype)), (M, out_dtype)
            assert bool((t[0] == -7).all()) and bool((t[-1] == -7).all()), (M, out_dtype)
        parts = partials(X[:M], W, leaf, k_first, 4)
        assert torch.equal(tb.tbik_tree_combine(parts, out_dtype=torch.float32), want[:M]), M
