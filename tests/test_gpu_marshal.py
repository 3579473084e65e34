"""The binding's common calls go through its native half (csrc/marshal.cpp), all others through ctypes: the two give the same bits, and an argument
that is not one of the common kind is answered (or refused) as ctypes answers it."""
import ctypes as C
import threading

import pytest
import torch

from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu
bf, f16, f32, u8 = torch.bfloat16, torch.float16, torch.float32, torch.uint8


def rnd(shape, dtype=bf):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(hash(shape) % 1000)
    return torch.randn(shape, generator=g, device="cuda:0").to(dtype)


def bits(shape, lo=0, hi=120):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(len(shape))
    return torch.randint(lo, hi, shape, generator=g, device="cuda:0", dtype=u8)


def scales(rows, K):
    return bits((rows, K // 32), 120, 130)


def cu(*v):
    return torch.tensor(v, dtype=torch.int32, device="cuda:0")


X, W, K, N = rnd, rnd, 1024, 256
CALLS = {
    "gemm": lambda m: (tb.tbik_gemm, (rnd((m, K)), rnd((K, N)), 128, 1)),
    "gemm_f16": lambda m: (tb.tbik_gemm_f16, (rnd((m, K), f16), rnd((K, N), f16), 128, 1, f32)),
    "gemm_f32": lambda m: (tb.tbik_gemm_f32, (rnd((m, K), f32), rnd((K, N), f32), 128, 1)),
    "partials": lambda m: (tb.tbik_gemm_shard_partials, (rnd((m, K)), rnd((K, N)), 128, 1, 4)),
    "partials_f32": lambda m: (tb.tbik_gemm_shard_partials_f32, (rnd((m, K), f32), rnd((K, N), f32), 128, 1, 2)),
    "swiglu": lambda m: (tb.tbik_gemm_swiglu, (rnd((m, K), f16), rnd((K, 2 * N), f16), 128, 1)),
    "fp8": lambda m: (tb.tbik_gemm_fp8, (bits((m, K)), bits((N, K)), 128, 1, "e5m2")),
    "mxfp8": lambda m: (tb.tbik_gemm_mxfp8, (bits((m, K)), scales(m, K), bits((N, K)), scales(N, K), 128, 1, "e4m3", f32)),
    "mxfp6": lambda m: (tb.tbik_gemm_mxfp6, (bits((m, K * 3 // 4)), scales(m, K), bits((N, K * 3 // 4)), scales(N, K), 256, 1, "e3m2")),
    "mxfp4": lambda m: (tb.tbik_gemm_mxfp4, (bits((m, K // 2)), scales(m, K), bits((N, K // 2)), scales(N, K), 256, 1)),
    "rmsnorm": lambda m: (tb.tbik_rmsnorm, (rnd((m, K)), rnd((K,)), 1e-6)),
    "combine": lambda m: (tb.tbik_combine_residual_rmsnorm_f16, (rnd((2, m, K), f32), rnd((m, K), f16), rnd((K,), f16), 1e-6)),
    "rows": lambda m: (tb.tbik_row_reduce, (rnd((m, 20000), f32), tb.TBIK_LOGSOFTMAX)),
    "row_max": lambda m: (tb.tbik_row_reduce, (rnd((m, 20000)), tb.TBIK_MAX)),
    "attention": lambda m: (tb.tbik_attention, (rnd((m, 8, 128)), rnd((m + 9, 2, 128)), rnd((m + 9, 2, 128)), cu(0, m), cu(0, m + 9), m, 128 ** -0.5, True, None, m + 9)),
}


@pytest.mark.parametrize("m", [1, 33, 130])
@pytest.mark.parametrize("name", list(CALLS))
def test_native_and_ctypes_give_the_same_bits(name, m, monkeypatch):
    f, args = CALLS[name](m)
    tb.lib()
    answers = []
    real = tb._native
    spy = lambda g: (lambda *a: answers.append(g(*a)) or answers[-1])
    monkeypatch.setattr(tb, "_native", type("Spy", (), {k: staticmethod(spy(getattr(real, k))) for k in ("product", "rmsnorm", "combine", "row_reduce", "attention")}))
    native = f(*args)
    assert len(answers) == 1 and answers[0] is not None           # a common call is answered there
    monkeypatch.setattr(tb, "_native", tb._NotLoaded)
    other = f(*args)
    for a, b in zip(native if isinstance(native, tuple) else (native,), other if isinstance(other, tuple) else (other,)):
        assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and not a.requires_grad
        assert torch.equal(a.view(u8), b.view(u8))


def test_uncommon_arguments_are_left_to_ctypes():
    tb.lib()
    n = tb._native
    g = tb._NUMBER["tbik_gemm"]
    x, w = rnd((4, K)), rnd((K, N))
    assert n.product(g, x, None, w, None, 128, 1, bf, 0) is not None
    class Sub(torch.Tensor):
        pass
    for bad in [(g, x.t().contiguous().t(), None, w, None, 128, 1, bf, 0), (g, x.to(f16), None, w, None, 128, 1, bf, 0), (g, x.cpu(), None, w, None, 128, 1, bf, 0),
                (g, x, None, w[:-1], None, 128, 1, bf, 0), (g, x, None, w, None, 128.0, 1, bf, 0), (g, x, None, w, None, 128, 1, torch.int32, 0),
                (g, x.as_subclass(Sub), None, w, None, 128, 1, bf, 0), (g, x[0], None, w, None, 128, 1, bf, 0), (g, x, None, w, None, 1 << 40, 1, bf, 0),
                (g, None, None, w, None, 128, 1, bf, 0), (99, x, None, w, None, 128, 1, bf, 0), (g, x, None, w)]:
        assert n.product(*bad) is None
    assert n.rmsnorm(tb._NUMBER["tbik_rmsnorm"], x, rnd((K,)), 0) is None and n.rmsnorm(tb._NUMBER["tbik_rmsnorm"], x[:, ::2], rnd((K // 2,)), 1e-6) is None
    # float8 tensors, integers as eps: answered through ctypes
    assert torch.equal(tb.tbik_gemm_fp8(bits((3, K)).view(torch.float8_e4m3fn), bits((N, K)).view(torch.float8_e4m3fn), 128).view(u8), tb.tbik_gemm_fp8(bits((3, K)), bits((N, K)), 128).view(u8))
    tb.tbik_rmsnorm(x, rnd((K,)), 0)


def test_errors_are_those_of_the_library():
    x, w = rnd((4, K)), rnd((K, N))
    tb.lib()
    with pytest.raises(tb.TbikError, match="tbik_gemm: "):
        tb.tbik_gemm(x, w, 100, 1)                                # a leaf that does not divide K
    with pytest.raises(tb.TbikError, match="tbik_gemm_shard_partials: "):
        tb.tbik_gemm_shard_partials(x, w, 128, 1, 3)
    with pytest.raises(KeyError):
        tb.tbik_gemm_fp8(bits((3, K)), bits((N, K)), 128, 1, "e9m9")
    with pytest.raises(AssertionError):
        tb.tbik_gemm(x, w[:-1], 128, 1)
    with pytest.raises(Exception):
        torch.vmap(lambda t: tb.tbik_gemm(t, w, 128, 1))(torch.stack([x, x]))


@pytest.mark.parametrize("name", ["gemm", "gemm_f16", "fp8", "mxfp8", "mxfp6", "mxfp4"])
def test_no_output_type_is_answered_as_ctypes_answers_it(name, monkeypatch):
    """out_dtype=None: torch's new_empty takes the operand's type, which the library has for 16 bits and not for bytes."""
    f, args = CALLS[name](5)
    args = args[:-1] if args[-1] is f32 else args

    def answer():
        try:
            return f(*args, out_dtype=None)
        except TypeError as e:
            return str(e)

    tb.lib()
    native = answer()
    monkeypatch.setattr(tb, "_native", tb._NotLoaded)
    other = answer()
    if name.startswith("gemm"):
        assert native.dtype == other.dtype == args[0].dtype and torch.equal(native.view(u8), other.view(u8))
    else:
        assert native == other and "uint8" in native


def test_another_stream_gets_a_workspace_of_its_own():
    x, w = rnd((33, 8 * K)), rnd((8 * K, N))
    want = tb.tbik_gemm(x, w, 128, 1)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = tb.tbik_gemm(x, w, 128, 1)
        mine = tb._ws_cache.get((0, s.cuda_stream))
    s.synchronize()
    assert torch.equal(got, want)
    assert tb.gemm_16bit_workspace_bytes(33, N, 8 * K, 128, 1) == 0 or mine is not None


FREE = 31                                                             # a number that no call of the library has


@pytest.mark.parametrize("cached", [True, False])
@pytest.mark.parametrize("kind", ["product", "row_reduce", "attention"])
def test_a_workspace_outlives_the_call_that_uses_it(kind, cached):
    """While a call is inside the library the interpreter lock is free, and another thread on the same stream may need a larger
    workspace.  A function that stands for the library plays that thread: the workspace that the call was given is not handed
    out again before the call is over.  No kernel runs."""
    tb.lib()
    need = 48 << 20                                                   # a block of its own in torch's allocator
    args = {"product": [C.c_void_p, C.c_int64, C.c_void_p, C.c_int64, C.c_void_p, C.c_int64] + [C.c_int] * 6,
            "row_reduce": [C.c_void_p, C.c_int, C.c_void_p, C.c_int, C.c_int, C.c_int64],
            "attention": [C.c_void_p] * 6 + [C.c_int] * 8 + [C.c_int64] * 4 + [C.c_float, C.c_int]}[kind]
    sizes = {"product": [C.c_int] * 5, "row_reduce": [C.c_int, C.c_int64, C.c_int], "attention": [C.c_int] * 5}[kind]
    seen = []

    def other_thread():
        tb._workspace(2 * need, torch.device("cuda:0"))
        seen.append({torch.empty(need, dtype=torch.uint8, device="cuda:0").data_ptr() for _ in range(2)})

    @C.CFUNCTYPE(C.c_int, *args, C.c_void_p, C.c_size_t, C.c_void_p)
    def call(*a):
        seen.append(a[-3])
        t = threading.Thread(target=other_thread)
        t.start()
        t.join()
        return 0

    query = C.CFUNCTYPE(C.c_size_t, *sizes)(lambda *a: need)
    address = lambda f: C.cast(f, C.c_void_p).value
    tb._native.register(FREE, {"product": 0, "row_reduce": 10, "attention": 11}[kind], address(call), address(query), bf)
    torch.cuda.synchronize()
    tb._ws_cache.clear()
    torch.cuda.empty_cache()
    if cached:
        tb._workspace(need, torch.device("cuda:0"))
    x = rnd((4, K))
    q = rnd((4, 2, 128))
    y = {"product": lambda: tb._native.product(FREE, x, None, rnd((K, N)), None, 128, 1, bf, 0),
         "row_reduce": lambda: tb._native.row_reduce(FREE, x, 0),
         "attention": lambda: tb._native.attention(FREE, q, q, q, cu(0, 4), cu(0, 4), 4, 0.1, True, 4)}[kind]()
    assert torch.is_tensor(y) and len(seen) == 2
    assert seen[0] and seen[0] not in seen[1]
