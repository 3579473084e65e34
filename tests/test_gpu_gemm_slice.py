"""GPU tests of the one-launch kernel for up to 32 rows of the low-bit formats: every output bit equal to the reference
kernel's (one summation order, whatever computes it), at the edges of what the kernel takes: rows around its two groups of
16, channels that do not fill a slice, more slices than compute units (the short ring), superleaves shorter and longer than
the ring, fewer superleaves than wavefronts and several per wavefront, strided operands, both outputs."""
import pytest
import torch

from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu

FORMATS = ["fp8 e4m3", "fp8 e5m2", "mxfp8 e4m3", "mxfp8 e5m2", "mxfp6 e2m3", "mxfp6 e3m2", "mxfp4 e2m1"]
# (K, leaf, k_first): one superleaf of one step (of the 4- and 6-bit formats), two superleaves, eight of three steps, 16, four per wavefront
TREES = [(256, 256, 1), (3072, 512, 3), (6144, 256, 3), (4096, 256, 1), (8192, 256, 1)]


@pytest.fixture(autouse=True)
def _reset_variant():
    yield
    tb.tbik_set_gemm_variant(tb.VARIANT_AUTO)


def _operands(kind, fmt, rows, K, pad, g):
    """Random patterns (no NaN, no infinity) and scales of 2^-5 .. 2^5, in rows of a stride of their own."""
    per = {"fp8": 32, "mxfp8": 32, "mxfp6": 24, "mxfp4": 16}[kind] * (K // 32)
    q = torch.randint(0, 256, (rows, per + pad), generator=g, device="cuda", dtype=torch.uint8)
    if kind in ("fp8", "mxfp8"):                     # exponents that keep every product and sum finite
        q = q & (0xBF if fmt == "e4m3" else 0xBB)
    s = torch.randint(122, 133, (rows, K // 32 + pad // 4), generator=g, device="cuda", dtype=torch.uint8)
    return q[:, :per], s[:, :K // 32]


def _both(kind, fmt, X, Xs, W, Ws, leaf, k_first, out_dtype, out):
    if kind == "fp8":
        return (tb.tbik_gemm_fp8(X, W, leaf, k_first, fmt, out=out), tb.tbik_gemm_reference_fp8(X, W, leaf, k_first, 1, fmt, out_dtype=out_dtype)[0])
    if kind == "mxfp8":
        return (tb.tbik_gemm_mxfp8(X, Xs, W, Ws, leaf, k_first, fmt, out=out),
                tb.tbik_gemm_reference_mxfp8(X, Xs, W, Ws, leaf, k_first, 1, fmt, out_dtype=out_dtype)[0])
    if kind == "mxfp6":
        return (tb.tbik_gemm_mxfp6(X, Xs, W, Ws, leaf, k_first, fmt, out=out),
                tb.tbik_gemm_reference_mxfp6(X, Xs, W, Ws, leaf, k_first, 1, fmt, out_dtype=out_dtype)[0])
    return (tb.tbik_gemm_mxfp4(X, Xs, W, Ws, leaf, k_first, out=out), tb.tbik_gemm_reference_mxfp4(X, Xs, W, Ws, leaf, k_first, 1, out_dtype=out_dtype)[0])


@pytest.mark.parametrize("tree", range(len(TREES)))
@pytest.mark.parametrize("name", FORMATS)
def test_few_rows_equal_the_reference_kernel(name, tree):
    kind, fmt = name.split()
    K, leaf, k_first = TREES[tree]
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * tree + len(name))
    for M, N, pad in ((1, 16, 0), (15, 40, 16), (16, 4104, 0), (17, 8, 32), (31, 131, 0), (32, 272, 16)):
        long_for_scaled_8_bit = kind == "mxfp8" and K == 8192 and M >= 31                     # tiles are the quicker way there
        assert tb.gemm_route(kind, M, N, K, leaf, k_first)[0][1] == ("tiles" if long_for_scaled_8_bit else "slices")
        X, Xs = _operands(kind, fmt, M, K, pad, g)
        W, Ws = _operands(kind, fmt, N, K, pad, g)
        for out_dtype in (torch.float32, torch.bfloat16):
            out = torch.full((M + 2, N + 3), -7.0, dtype=out_dtype, device="cuda")
            y, want = _both(kind, fmt, X, Xs, W, Ws, leaf, k_first, out_dtype, out[1:M + 1, :N])
            assert torch.equal(y.contiguous().view(torch.uint8), want.view(torch.uint8)), (M, N, out_dtype)
            assert bool((out[0] == -7).all()) and bool((out[M + 1] == -7).all()) and bool((out[:, N:] == -7).all()), (M, N)


# (kind, K, leaf, rows): 64 and 128 superleaves, eight and sixteen per wavefront: every level of a wavefront's own tree
DEEP = [("fp8 e4m3", 8192, 128, (1, 16, 17, 32)), ("fp8 e4m3", 16384, 128, (1, 16, 17, 32)), ("fp8 e5m2", 16384, 128, (16, 17)),
        ("mxfp8 e4m3", 8192, 128, (1, 16, 17, 32)), ("mxfp8 e4m3", 16384, 128, (1, 16)), ("mxfp6 e2m3", 16384, 256, (16, 17)),
        ("mxfp6 e3m2", 32768, 256, (1, 16, 17)), ("mxfp4 e2m1", 16384, 256, (16, 17)), ("mxfp4 e2m1", 32768, 256, (1, 16))]


@pytest.mark.parametrize("name,K,leaf,rows", DEEP)
def test_many_superleaves_equal_the_reference_kernel(name, K, leaf, rows):
    kind, fmt = name.split()
    g = torch.Generator(device="cuda")
    g.manual_seed(K + len(name))
    N = 4093
    W, Ws = _operands(kind, fmt, N, K, 0, g)
    X, Xs = _operands(kind, fmt, max(rows), K, 0, g)
    for M in rows:
        assert tb.gemm_route(kind, M, N, K, leaf) == [(M, "slices", 0, 0)]
        out = torch.full((M + 2, N + 3), -7.0, dtype=torch.float32, device="cuda")
        y, want = _both(kind, fmt, X[:M], Xs[:M], W, Ws, leaf, 1, torch.float32, out[1:M + 1, :N])
        assert torch.equal(y.contiguous().view(torch.uint8), want.view(torch.uint8)), M
        assert bool((out[0] == -7).all()) and bool((out[M + 1] == -7).all()) and bool((out[:, N:] == -7).all()), M


@pytest.mark.parametrize("name,K,leaf", [("fp8 e4m3", 32768, 128), ("mxfp8 e5m2", 32768, 128), ("mxfp6 e2m3", 65536, 256), ("mxfp4 e2m1", 65536, 256)])
def test_more_superleaves_than_a_wavefront_holds_go_to_tiles(name, K, leaf):
    """256 superleaves would be 32 per wavefront."""
    kind, fmt = name.split()
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    M, N = 5, 264
    assert tb.gemm_route(kind, M, N, K, leaf)[0][1] == "tiles"
    (W, Ws), (X, Xs) = _operands(kind, fmt, N, K, 0, g), _operands(kind, fmt, M, K, 0, g)
    out = torch.full((M, N), -7.0, dtype=torch.float32, device="cuda")
    y, want = _both(kind, fmt, X, Xs, W, Ws, leaf, 1, torch.float32, out)
    assert torch.equal(y.view(torch.uint8), want.view(torch.uint8))
