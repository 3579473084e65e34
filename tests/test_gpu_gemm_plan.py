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
        ws = torch.full((max(256, tb.gemm_16bit_workspace_bytes(M, N, K, LEAF, 1)) // 4,), float("nan"), dtype=torch.float32, device="cuda:0")
        assert torch.equal(call(X, W, LEAF, 1, out_dtype=torch.float32, workspace=ws).view(torch.int32), want)
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
    """A batch a little above full rounds of 128-row tiles, which 16-bit operands (and MXFP6 at 1 and 4 rows more, whose last
    piece goes to slices) compute in two pieces here: rows equal those of other batch sizes."""
    Kp, Np = 2048, 1024                                           # 8 column tiles: 32 row tiles fill a round
    pieces = {kind: len(tb.gemm_route(kind, M, Np, Kp, LEAF, 1)) for kind in ("bf16", "mxfp8", "mxfp4", "mxfp6")}
    assert pieces == {"bf16": 2, "mxfp8": 1, "mxfp4": 1, "mxfp6": 2 if M <= 4100 else 1}
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


def layer(kind, M, Kl, Nl, seed):
    """Operands of a [M, Kl] x [Kl, Nl] product made of 300 different rows and 500 different columns (neither a multiple of a
    tile), the call, its reference kernel's fp32 result, the workspace size and the re-tiled scales' part of it."""
    rep = lambda t, n: t.repeat(-(-n // t.shape[0]), 1)[:n].contiguous()
    if kind in ("bf16", "fp16"):
        dt, sfx = (torch.bfloat16, "") if kind == "bf16" else (torch.float16, "_f16")
        g = torch.Generator(device="cuda:0")
        g.manual_seed(seed)
        ops = [torch.randn((M, Kl), generator=g, device="cuda:0").to(dt), (torch.randn((Kl, Nl), generator=g, device="cuda:0") * 0.02).to(dt)]
        call, ref, need = getattr(tb, "tbik_gemm" + sfx), getattr(tb, "tbik_gemm_reference" + sfx), tb.gemm_16bit_workspace_bytes
        return ops, call, (lambda *a: ref(*a, out_dtype=torch.float32)[1]), need, 0
    host = getattr(syn, "gemm_random_" + kind)(seed, 300, Kl, 500)
    if kind == "fp8":
        host = (host[0], host[1].T)
    dev = [torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0") for t in host]
    half = len(dev) // 2
    ops = [rep(t, M) for t in dev[:half]] + [rep(t, Nl) for t in dev[half:]]
    ref = getattr(tb, "tbik_gemm_reference_" + kind)
    scales = 0 if kind == "fp8" or M < 128 else getattr(tb, "gemm_%s_workspace_bytes" % kind)(M, Nl, 256, 256, 1) * (Kl // 256)     # (K = one superleaf is never split)
    return ops, getattr(tb, "tbik_gemm_" + kind), (lambda *a: ref(*a)[0]), getattr(tb, "gemm_%s_workspace_bytes" % kind), scales


def padded(M, Nl, dtype):
    """An output with eight more columns of sevens than the call may write."""
    buf = torch.full((M, Nl + 8), 7.0, dtype=dtype, device="cuda:0")
    return buf, buf[:, :Nl]


@pytest.mark.parametrize("kind,out_dtypes", [("bf16", (torch.bfloat16, torch.float32)), ("fp16", (torch.float16, torch.float32)),
                                             ("fp8", (torch.bfloat16, torch.float32)), ("mxfp8", (torch.bfloat16, torch.float32)),
                                             ("mxfp6", (torch.bfloat16, torch.float32)), ("mxfp4", (torch.bfloat16, torch.float32))])
@pytest.mark.parametrize("M,rest_planes", [(1025, 8), (1057, 8), (1152, (8, 4)), (1160, 4), (2200, 4)])
def test_both_pieces_of_a_cut_batch(kind, out_dtypes, M, rest_planes):
    """K = 12288: every format cuts these batches behind 1024 or 2048 rows.  The size that a call asks for shows it: planes of the
    last rows alone (and the microscaling formats' re-tiled scales of the whole call).  128 and 136 last rows re-tile once more,
    over the first piece's scales; 1, 33 and 152 are other heights and splits.  Every row against the reference kernel."""
    Kl, Nl, leaf, kf = 12288, 4096, 256, 3
    ops, call, ref, need, scales = layer(kind, M, Kl, Nl, M)
    rest = M % 1024
    full = need(M, Nl, Kl, leaf, kf)
    assert full - scales in [p * rest * Nl * 4 for p in np.atleast_1d(rest_planes)]
    want = ref(*ops, leaf, kf)
    for dt in out_dtypes:
        buf, out = padded(M, Nl, dt)
        ws = torch.full((full // 4,), float("nan"), dtype=torch.float32, device="cuda:0")
        call(*ops, leaf, kf, out=out, workspace=ws)
        bits = torch.int32 if dt == torch.float32 else torch.int16
        assert torch.equal(out.contiguous().view(bits), want.to(dt).view(bits)), dt
        assert (buf[:, Nl:] == 7.0).all()


@pytest.mark.parametrize("kind,M,Kl,leaf,kf,rule", [("bf16", 321, 12288, 256, 3, 1), ("fp16", 400, 12288, 256, 3, 1), ("mxfp8", 321, 12288, 256, 3, 1),
                                                    ("mxfp6", 385, 12288, 256, 3, 1), ("bf16", 1152, 12288, 256, 3, 1), ("fp8", 1152, 12288, 256, 3, 1),
                                                    ("mxfp4", 1057, 12288, 256, 3, 1), ("mxfp8", 1152, 12288, 256, 3, 1), ("bf16", 128, 12288, 256, 3, 8)])
def test_workspace_of_the_older_rule_alone(kind, M, Kl, leaf, kf, rule):
    """The planes of the older rule's split (`rule`; none for 1) are what a call insists on: the plan that fits them gives the
    same bits, as do a size between it and the advertised one, and the advertised one; 256 bytes less are refused."""
    Nl = 4096
    ops, call, ref, need, scales = layer(kind, M, Kl, Nl, M)
    full, least = need(M, Nl, Kl, leaf, kf), scales + (rule * M * Nl * 4 if rule > 1 else 0)
    assert least < full or rule > 1
    want = ref(*ops, leaf, kf).view(torch.int32)
    for nbytes in sorted({least, (least + full) // 512 * 256, full}):
        ws = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda:0")
        got = call(*ops, leaf, kf, out_dtype=torch.float32, workspace=ws)
        assert torch.equal(got.view(torch.int32), want), nbytes
    if least:
        with pytest.raises(tb.TbikError):
            call(*ops, leaf, kf, workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda:0"))


def test_a_16_bit_call_holds_no_planes_of_the_fp32_plans(monkeypatch):
    """600 rows of 4096 x 4096: no planes in 16 bits, 75 MiB in fp32."""
    asked = []
    tb.lib()
    tb._ws_cache.clear()                                              # what is there is taken without asking
    monkeypatch.setattr(tb, "_workspace", lambda nbytes, device, real=tb._workspace: asked.append(nbytes) or real(nbytes, device))
    for dt, call, parts in ((torch.bfloat16, tb.tbik_gemm, tb.tbik_gemm_shard_partials), (torch.float16, tb.tbik_gemm_f16, tb.tbik_gemm_shard_partials_f16)):
        X, W = torch.ones((600, 4096), dtype=dt, device="cuda:0"), torch.ones((4096, 4096), dtype=dt, device="cuda:0")
        assert (call(X, W, 256, 1) == 4096).all() and (parts(X, W, 256, 1, 2) == 2048).all()
    assert asked == []
    assert (tb.tbik_gemm_f32(torch.ones((600, 4096), device="cuda:0"), torch.ones((4096, 4096), device="cuda:0"), 256, 1) == 4096).all()
    assert asked and min(asked) >= 600 * 4096 * 4                     # a call that needs planes asks here
