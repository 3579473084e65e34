"""Whatever tile height and K split the time model chooses for 16-, 8-, 6- and 4-bit operands, a call gives the bits of the
reference kernel (0 differing bits), at batch sizes around the edges of the tile heights and of rounds of 256 work items;
also with a workspace that holds only the planes of the older rule's split, or nothing but what the call insists on."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2511_17826_amd import binding as tb
from paper_2511_17826_amd import synthetic as syn

pytestmark = pytest.mark.gpu

K, N, LEAF = 2048, 1536, 256


@pytest.mark.parametrize("M", [1, 31, 33, 64, 65, 97, 129, 200, 300, 700])
def test_16_bit(M):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(M)
    for dt, call, ref, partials in ((torch.bfloat16, tb.tbik_gemm, tb.tbik_gemm_reference, tb.tbik_gemm_shard_partials),
                                    (torch.float16, tb.tbik_gemm_f16, tb.tbik_gemm_reference_f16, tb.tbik_gemm_shard_partials_f16)):
        X = torch.randn((M, K), generator=g, device="cuda:0").to(dt)
        W = (torch.randn((K, N), generator=g, device="cuda:0") * 0.02).to(dt)
        want = ref(X, W, LEAF, 1, out_dtype=torch.float32)[1].view(torch.int32)
        assert torch.equal(call(X, W, LEAF, 1, out_dtype=torch.float32).view(torch.int32), want)
        full, done = tb.gemm_workspace_bytes(M, N, K, LEAF, 1), 0
        for planes in (8, 4, 2, 1):
            if planes * M * N * 4 > full:
                continue
            ws = torch.full((planes * M * N,), float("nan"), dtype=torch.float32, device="cuda:0")
            try:
                out = call(X, W, LEAF, 1, out_dtype=torch.float32, workspace=ws)
            except tb.TbikError:
                continue
            done += 1
            assert torch.equal(out.view(torch.int32), want), planes
        for P in (1, 2, 8):
            assert torch.equal(tb.tbik_tree_combine(partials(X, W, LEAF, 1, P), out_dtype=torch.float32).view(torch.int32), want), P


@pytest.mark.parametrize("kind", ["fp8", "mxfp8", "mxfp6", "mxfp4"])
@pytest.mark.parametrize("M", [1, 33, 65, 100, 129, 300, 700])
def test_low_bit(kind, M):
    if kind == "fp8":
        X, W = syn.gemm_random_fp8(M, M, K, N)
        ops = (X, W.T)                                            # the calls take the transposed weight
        dev = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in ops]
        call, ref, parts, need = tb.tbik_gemm_fp8, tb.tbik_gemm_reference_fp8, tb.tbik_gemm_shard_partials_fp8, tb.gemm_fp8_workspace_bytes
    else:
        ops = getattr(syn, "gemm_random_" + kind)(M, M, K, N, scale_spread=2)
        dev = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in ops]
        call, ref, parts, need = (getattr(tb, n % kind) for n in ("tbik_gemm_%s", "tbik_gemm_reference_%s", "tbik_gemm_shard_partials_%s",
                                                                  "gemm_%s_workspace_bytes"))
    want = ref(*dev, LEAF, 1)[0].view(torch.int32)
    assert torch.equal(call(*dev, LEAF, 1, out_dtype=torch.float32).view(torch.int32), want)
    ws = torch.full((max(256, need(M, N, K, LEAF, 1)) // 4,), float("nan"), dtype=torch.float32, device="cuda:0")
    assert torch.equal(call(*dev, LEAF, 1, out_dtype=torch.float32, workspace=ws).view(torch.int32), want)
    for P in (2, 8):
        assert torch.equal(tb.tbik_tree_combine(parts(*dev, LEAF, 1, P), out_dtype=torch.float32).view(torch.int32), want), P


@pytest.mark.parametrize("M", [4097, 4100, 4224, 4300])
def test_last_rows_as_a_call_of_their_own(M):
    """A batch a little above full rounds of 128-row tiles is computed in two pieces: rows equal those of other batch sizes."""
    Kp, Np = 2048, 1024                                           # 8 column tiles: 32 row tiles fill a round
    g = torch.Generator(device="cuda:0")
    g.manual_seed(M)
    X = torch.randn((M, Kp), generator=g, device="cuda:0").to(torch.bfloat16)
    W = (torch.randn((Kp, Np), generator=g, device="cuda:0") * 0.02).to(torch.bfloat16)
    want = tb.tbik_gemm(X[-700:], W, LEAF, 1)
    head = tb.tbik_gemm(X[:700], W, LEAF, 1)
    got = tb.tbik_gemm(X, W, LEAF, 1)
    assert torch.equal(got[-700:].view(torch.int16), want.view(torch.int16)) and torch.equal(got[:700].view(torch.int16), head.view(torch.int16))
    whole = tb.tbik_gemm_reference(X, W, LEAF, 1, out_dtype=torch.bfloat16)[1]
    assert torch.equal(got.view(torch.int16), whole.view(torch.int16))
    for kind in ("mxfp8", "mxfp4", "mxfp6"):
        ops = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in getattr(syn, "gemm_random_" + kind)(M, 300, Kp, Np)]
        rep = -(-M // 300)
        dev = [ops[0].repeat(rep, 1)[:M].contiguous(), ops[1].repeat(rep, 1)[:M].contiguous(), ops[2], ops[3]]
        y = getattr(tb, "tbik_gemm_" + kind)(*dev, LEAF, 1)
        one = getattr(tb, "tbik_gemm_" + kind)(*ops, LEAF, 1)
        assert torch.equal(y.view(torch.int16), one.repeat(rep, 1)[:M].view(torch.int16)), kind


def test_a_16_bit_call_holds_no_planes_of_the_fp32_plans(monkeypatch):
    """600 rows of 4096 x 4096: no planes in 16 bits, 75 MiB in fp32."""
    asked = []
    monkeypatch.setattr(tb, "_workspace", lambda nbytes, device, real=tb._workspace: asked.append(nbytes) or real(nbytes, device))
    for dt, call, parts in ((torch.bfloat16, tb.tbik_gemm, tb.tbik_gemm_shard_partials), (torch.float16, tb.tbik_gemm_f16, tb.tbik_gemm_shard_partials_f16)):
        X, W = torch.ones((600, 4096), dtype=dt, device="cuda:0"), torch.ones((4096, 4096), dtype=dt, device="cuda:0")
        assert (call(X, W, 256, 1) == 4096).all() and (parts(X, W, 256, 1, 2) == 2048).all()
    assert asked == []
