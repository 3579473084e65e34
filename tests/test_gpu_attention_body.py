"""attention_kernel's main loop takes two key tiles at a time, with the scores of the next tile formed beside the softmax step
of this one; masked tiles, a wavefront's last ones and those around the end of a split take another way.  Its rows have the
bits of the kernel for few queries (one query at a time over the keys it sees) at every parity of the tiles involved."""
import pytest
import torch

from paper_2511_17826_amd import binding as tb
from test_gpu_attention import i32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("Lq,Lk", [(63, 63), (64, 64), (65, 65), (129, 129), (40, 191), (97, 192), (200, 193), (33, 257), (130, 449),
                                   (70, 4096), (100, 4097), (65, 4160), (66, 4225), (130, 8257)])
def test_rows_are_those_of_single_queries(Lq, Lk, dtype):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(Lq * 10007 + Lk)
    rnd = lambda n, h: torch.randn((n, h, 128), generator=g, device="cuda:0").to(dtype)
    Q, K, V = rnd(Lq, 8), rnd(Lk, 2), rnd(Lk, 2)
    call = tb.tbik_attention if dtype == torch.bfloat16 else tb.tbik_attention_f16
    O = call(Q, K, V, i32([0, Lq]), i32([0, Lk]), Lq, 128 ** -0.5, True, max_seqlen_k=Lk)
    for r in sorted({0, 1, 31, 32, min(33, Lq - 1), Lq // 2, Lq - 2, Lq - 1}):
        sees = Lk - Lq + r + 1
        if sees <= 0:
            assert not O[r].any(), r                              # a query that sees no key
            continue
        one = call(Q[r:r + 1], K[:sees], V[:sees], i32([0, 1]), i32([0, sees]), 1, 128 ** -0.5, True, max_seqlen_k=sees)
        assert torch.equal(O[r].view(torch.int16), one[0].view(torch.int16)), r
