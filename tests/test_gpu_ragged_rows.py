"""GPU tests of the ragged last row tile of the tiled GEMM kernels (16-bit, 8-bit, MXFP8, MXFP6, MXFP4): every bit equal to the
reference kernel's and nothing written past the last row, at one row past a tile, one row short of one, block rows of 32 that are
full, short and absent, at every tile height, for 16-bit, fp32 and shard-partial outputs and the gated activation."""
import pytest
import torch

from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu
K, N, LEAF = 1024, 256, 256
HEIGHTS = {128: tb.VARIANT_T128, 64: tb.VARIANT_T64, 32: tb.VARIANT_T32}
ROWS = [1, 31, 32, 33, 63, 65, 95, 97, 127, 129, 160, 191, 223, 255]


@pytest.fixture(autouse=True)
def _reset_variant():
    yield
    tb.tbik_set_gemm_variant(tb.VARIANT_AUTO)


def _framed(rows, cols, dtype):
    """A tensor with guard rows around the view that a call may write."""
    t = torch.full((rows + 2, cols), -7.0, dtype=dtype, device="cuda")
    return t, t[1:rows + 1]


def _guards_untouched(t):
    return bool((t[0] == -7).all()) and bool((t[-1] == -7).all())


def _equal(a, b):
    return torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))


def _low_bit(kind, rows, g):
    per = {"fp8": 32, "mxfp8": 32, "mxfp6": 24, "mxfp4": 16}[kind] * (K // 32)
    q = torch.randint(0, 256, (rows, per), generator=g, device="cuda", dtype=torch.uint8)
    if kind in ("fp8", "mxfp8"):
        q &= 0xBF                                    # E4M3 without NaN
    return q, torch.randint(122, 133, (rows, K // 32), generator=g, device="cuda", dtype=torch.uint8)


@pytest.mark.parametrize("height", sorted(HEIGHTS))
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_16bit(dtype, height):
    g = torch.Generator(device="cuda")
    g.manual_seed(height)
    f16 = dtype == torch.float16
    gemm, ref = (tb.tbik_gemm_f16, tb.tbik_gemm_reference_f16) if f16 else (tb.tbik_gemm, tb.tbik_gemm_reference)
    partials = tb.tbik_gemm_shard_partials_f16 if f16 else tb.tbik_gemm_shard_partials
    W = torch.randn((K, N), generator=g, device="cuda").to(dtype)
    for M in ROWS:
        X = torch.randn((M, K), generator=g, device="cuda").to(dtype)
        want = ref(X, W, LEAF, 1, 1, out_dtype=torch.float32)[1]
        tb.tbik_set_gemm_variant(HEIGHTS[height])
        for out_dtype in (dtype, torch.float32):
            t, view = _framed(M, N, out_dtype)
            gemm(X, W, LEAF, 1, out=view)
            assert _equal(view, want.to(out_dtype)) and _guards_untouched(t), (M, out_dtype)
        t = torch.full((2 * M + 2, N), -7.0, device="cuda")
        parts = partials(X, W, LEAF, 1, 2, out=t[1:2 * M + 1].view(2, M, N))
        assert _equal(tb.tbik_tree_combine(parts, out_dtype=torch.float32), want) and _guards_untouched(t), M
        tb.tbik_set_gemm_variant(tb.VARIANT_AUTO)
        if height == 128:
            t, view = _framed(M, N // 2, dtype)
            tb.tbik_gemm_swiglu(X, W, LEAF, 1, out=view)
            gu = want.to(dtype)
            assert _equal(view, tb.tbik_silu_mul(gu[:, :N // 2], gu[:, N // 2:])) and _guards_untouched(t), M


@pytest.mark.parametrize("height", sorted(HEIGHTS))
@pytest.mark.parametrize("kind", ["fp8", "mxfp8", "mxfp6", "mxfp4"])
def test_low_bit(kind, height):
    g = torch.Generator(device="cuda")
    g.manual_seed(height)
    W, Ws = _low_bit(kind, N, g)
    for M in ROWS:
        X, Xs = _low_bit(kind, M, g)
        if kind == "fp8":
            gemm = lambda out: tb.tbik_gemm_fp8(X, W, LEAF, 1, out=out)
            want = tb.tbik_gemm_reference_fp8(X, W, LEAF, 1)[0]
        elif kind == "mxfp8":
            gemm = lambda out: tb.tbik_gemm_mxfp8(X, Xs, W, Ws, LEAF, 1, out=out)
            want = tb.tbik_gemm_reference_mxfp8(X, Xs, W, Ws, LEAF, 1)[0]
        elif kind == "mxfp6":
            gemm = lambda out: tb.tbik_gemm_mxfp6(X, Xs, W, Ws, LEAF, 1, out=out)
            want = tb.tbik_gemm_reference_mxfp6(X, Xs, W, Ws, LEAF, 1)[0]
        else:
            gemm = lambda out: tb.tbik_gemm_mxfp4(X, Xs, W, Ws, LEAF, 1, out=out)
            want = tb.tbik_gemm_reference_mxfp4(X, Xs, W, Ws, LEAF, 1)[0]
        tb.tbik_set_gemm_variant(HEIGHTS[height])
        for out_dtype in (torch.bfloat16, torch.float32):
            t, view = _framed(M, N, out_dtype)
            gemm(view)
            assert _equal(view, want.to(out_dtype)) and _guards_untouched(t), (M, out_dtype)
        tb.tbik_set_gemm_variant(tb.VARIANT_AUTO)


@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("kind", ["bf16", "fp8", "mxfp8", "mxfp6", "mxfp4"])
def test_output_rows_far_apart(kind, out_dtype):
    """Output rows so far apart that an offset inside the tile passes 32 bits."""
    M = 31
    ld = 72_000_000 if out_dtype == torch.bfloat16 else 36_000_000                  # the last row begins 4.32 GB on
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    out = torch.empty((M - 1) * ld + N, dtype=out_dtype, device="cuda").as_strided((M, N), (ld, 1))
    out.fill_(-7.0)
    if kind == "bf16":
        X = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
        W = torch.randn((K, N), generator=g, device="cuda").to(torch.bfloat16)
        want = tb.tbik_gemm_reference(X, W, LEAF, 1, 1, out_dtype=torch.float32)[1]
        gemm = lambda: tb.tbik_gemm(X, W, LEAF, 1, out=out)
    else:
        (X, Xs), (W, Ws) = _low_bit(kind, M, g), _low_bit(kind, N, g)
        args = (X, W) if kind == "fp8" else (X, Xs, W, Ws)
        want = getattr(tb, "tbik_gemm_reference_" + kind)(*args, LEAF, 1)[0]
        gemm = lambda: getattr(tb, "tbik_gemm_" + kind)(*args, LEAF, 1, out=out)
    for variant in (tb.VARIANT_T32, tb.VARIANT_T64, tb.VARIANT_T128, tb.VARIANT_AUTO):
        tb.tbik_set_gemm_variant(variant)
        out.fill_(-7.0)
        gemm()
        assert _equal(out, want.to(out_dtype)), variant
