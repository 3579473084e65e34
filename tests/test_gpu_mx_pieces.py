"""GPU test of microscaling GEMMs whose batch is cut into two pieces that share one re-tiling of the scales: every bit equal to
the reference kernel's, with last pieces below and above 128 rows, of tiles lower than the 128 rows the scales are re-tiled in,
and in a workspace of exactly the size asked for, filled with other bytes before the call."""
import pytest
import torch

from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,M,K,N,leaf,k_first", [
    ("mxfp8", 1060, 4096, 4096, 256, 1), ("mxfp8", 1300, 12288, 4096, 256, 3), ("mxfp8", 1500, 12288, 4096, 256, 3),
    ("mxfp4", 1300, 12288, 4096, 256, 3), ("mxfp4", 1500, 12288, 4096, 256, 3), ("mxfp4", 1100, 4096, 4096, 256, 1),
    ("mxfp4", 800, 4096, 6144, 256, 1), ("mxfp6", 2200, 4096, 4096, 256, 1), ("mxfp6", 1300, 12288, 4096, 256, 3)])
def test_pieces_equal_the_reference_kernel(kind, M, K, N, leaf, k_first):
    pieces = tb.gemm_route(kind, M, N, K, leaf, k_first)
    assert len(pieces) == 2 and all(p[1] == "tiles" for p in pieces)
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    per = {"mxfp8": 32, "mxfp6": 24, "mxfp4": 16}[kind] * (K // 32)

    def operand(rows):
        q = torch.randint(0, 256, (rows, per), generator=g, device="cuda", dtype=torch.uint8)
        return q & 0xBF if kind == "mxfp8" else q, torch.randint(122, 133, (rows, K // 32), generator=g, device="cuda", dtype=torch.uint8)

    X, Xs = operand(M)
    W, Ws = operand(N)
    need = int(getattr(tb.lib(), "tbik_gemm_%s_workspace_bytes" % kind)(M, N, K, leaf, k_first))
    ws = torch.randint(0, 256, (need,), generator=g, device="cuda", dtype=torch.uint8)
    gemm = getattr(tb, "tbik_gemm_" + kind)
    want = getattr(tb, "tbik_gemm_reference_" + kind)(X, Xs, W, Ws, leaf, k_first)[0]
    for out_dtype in (torch.float32, torch.bfloat16):
        y = gemm(X, Xs, W, Ws, leaf, k_first, out_dtype=out_dtype, workspace=ws)
        assert torch.equal(y.view(torch.uint8), want.to(out_dtype).view(torch.uint8)), out_dtype
