// The Python binding's common calls, marshalled natively: tensors in, one C call of libtbik, the new output tensor out.
//
// A call on a few rows is over on the GPU before Python has issued it.  Host time of a call through ctypes -> here, its launches (2.2 us
// each) included: 1 x 4096 x 4096 in bf16, two launches, 9.95 -> 6.9 us, in 8 bits, one, 8.0 -> 4.0; RMSNorm of a row 5.3 -> 4.0, attention
// of two short sequences 10.2 -> 4.4.  What a function below returns:
//   the output tensor(s), or an int: the library's status where it is not TBIK_OK, or None: "not one of the common calls" --
// an argument of another type, a view it would refuse, a tensor subclass, anything odd.  The caller then takes the way
// through ctypes, which answers every call as it always did, its errors included.  Nothing is decided here and nothing is kept between calls
// but the entry points' addresses; scratch memory comes from the binding's own cache of workspaces, by device and stream.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <climits>
#include <cstdint>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "tbik.h"

namespace {

enum Kind { GEMM, GEMM_F32, PARTIALS, PARTIALS_F32, SWIGLU, FP8, MX, MXFP4, RMSNORM, COMBINE, ROWS, ATTENTION, KINDS };
struct Entry {
    int kind = -1;
    void *call = nullptr, *need = nullptr;      // the C entry point and its workspace query
    at::ScalarType dtype = at::kFloat;          // of its operands
};
constexpr int MAX_ENTRIES = 32;
Entry entries[MAX_ENTRIES];                     // written while the library is loaded, under the interpreter lock
PyObject *workspaces = nullptr;                 // the binding's dict: (device index, stream) -> uint8 tensor
PyObject *make_workspace = nullptr;             // the binding's function that fills it

// A plain strided GPU tensor: no subclass, no wrapper of a transform, real sizes and memory.
const at::Tensor *plain(PyObject *o, int dim) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    const auto *impl = t.unsafeGetTensorImpl();
    const auto keys = t.key_set();
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.dim() != dim || impl->has_symbolic_sizes_strides() ||
        keys.has(c10::DispatchKey::Python) || keys.has(c10::DispatchKey::Functionalize) || keys.has(c10::DispatchKey::FuncTorchBatched) ||
        keys.has(c10::DispatchKey::FuncTorchGradWrapper) || keys.has(c10::DispatchKey::Conjugate) || keys.has(c10::DispatchKey::Negative))
        return nullptr;
    return &t;
}
const at::Tensor *matrix(PyObject *o, at::ScalarType dtype) {
    const at::Tensor *t = plain(o, 2);
    return t && t->scalar_type() == dtype && t->stride(1) == 1 && t->size(0) <= INT_MAX && t->size(1) <= INT_MAX ? t : nullptr;
}
bool integer(PyObject *o, int *v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long x = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || x < INT_MIN || x > INT_MAX) return false;
    *v = (int)x;
    return true;
}
bool number(PyObject *o, float *v) {
    if (!PyFloat_CheckExact(o)) return false;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
int type_code(at::ScalarType t) { return t == at::kFloat ? TBIK_F32 : t == at::kBFloat16 ? TBIK_BF16 : t == at::kHalf ? TBIK_F16 : -1; }

// Undefined unless it is a real tensor (a dispatch mode may hand out something else).
at::Tensor output(at::IntArrayRef sizes, const at::Tensor &like, at::ScalarType dtype) {
    at::Tensor t = at::empty(sizes, like.options().dtype(dtype).requires_grad(false));
    const auto keys = t.key_set();
    return t.is_cuda() && t.has_storage() && !keys.has(c10::DispatchKey::Python) ? t : at::Tensor();
}

// torch's current stream on the current device, as the binding passes it.
void *current_stream() { return (void *)c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream(); }

// Holds its tensor: while the interpreter lock is released another thread may put a larger one into the dict, and the
// allocator would give this one's memory away before the call's kernels are queued.
struct Room {
    at::Tensor held;
    void *at = nullptr;
    size_t bytes = 0;
    void take(const at::Tensor &ws) {
        held = ws;
        at = held.data_ptr();
        bytes = (size_t)held.numel();
    }
};
// The workspace of `need` bytes for `like`'s device and this stream; false: an error is set.
bool room_for(size_t need, PyObject *like, const at::Tensor &t, void *stream, Room *room) {
    if (need == 0) return true;
    PyObject *key = Py_BuildValue("(iK)", (int)t.device().index(), (unsigned long long)(uintptr_t)stream);
    if (!key) return false;
    PyObject *w = PyDict_GetItemWithError(workspaces, key);       // borrowed
    Py_DECREF(key);
    if (!w && PyErr_Occurred()) return false;
    if (w && THPVariable_Check(w)) {
        const at::Tensor &ws = THPVariable_Unpack(w);
        if ((size_t)ws.numel() >= need) {
            room->take(ws);
            return true;
        }
    }
    PyObject *device = PyObject_GetAttrString(like, "device");
    if (!device) return false;
    PyObject *made = PyObject_CallFunction(make_workspace, "KO", (unsigned long long)need, device);
    Py_DECREF(device);
    if (!made) return false;
    room->take(THPVariable_Unpack(made));
    Py_DECREF(made);
    return true;
}

#define UNCOMMON Py_RETURN_NONE
PyObject *wrapped(at::Tensor t, int status) { return status == 0 ? THPVariable_Wrap(std::move(t)) : PyLong_FromLong(status); }
const Entry *entry_of(PyObject *o, int kind_from, int kind_to) {
    int i;
    if (!integer(o, &i) || i < 0 || i >= MAX_ENTRIES || entries[i].kind < kind_from || entries[i].kind > kind_to) return nullptr;
    return &entries[i];
}

// Entries are called through the types that tbik.h declares for them; those of one kind have one type.
#define SAME(a, b) static_assert(std::is_same<decltype(&a), decltype(&b)>::value, #a " and " #b)
SAME(tbik_gemm, tbik_gemm_f16);
SAME(tbik_gemm, tbik_gemm_swiglu);
SAME(tbik_gemm_shard_partials, tbik_gemm_shard_partials_f16);
SAME(tbik_gemm_shard_partials, tbik_gemm_shard_partials_f32);
SAME(tbik_gemm_mxfp8, tbik_gemm_mxfp6);
SAME(tbik_rmsnorm, tbik_rmsnorm_f16);
SAME(tbik_combine_residual_rmsnorm, tbik_combine_residual_rmsnorm_f16);
SAME(tbik_attention, tbik_attention_f16);
SAME(tbik_gemm_16bit_workspace_bytes, tbik_gemm_f32_workspace_bytes);
SAME(tbik_gemm_16bit_workspace_bytes, tbik_gemm_swiglu_workspace_bytes);
SAME(tbik_gemm_16bit_workspace_bytes, tbik_gemm_fp8_workspace_bytes);
SAME(tbik_gemm_16bit_workspace_bytes, tbik_gemm_mxfp8_workspace_bytes);
SAME(tbik_gemm_16bit_workspace_bytes, tbik_gemm_mxfp6_workspace_bytes);
SAME(tbik_gemm_16bit_workspace_bytes, tbik_gemm_mxfp4_workspace_bytes);
SAME(tbik_gemm_16bit_workspace_bytes, tbik_attention_workspace_bytes);
#undef SAME
#define CALL(name) ((decltype(&name))e->call)
#define NEED(name) ((decltype(&name))e->need)
typedef void *P;
typedef int64_t L;

// product(entry, X, Xs, W, Ws, leaf, k_first, out dtype (None where the kind has one of its own), format or shards)
PyObject *product(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 9) UNCOMMON;
    const Entry *e = entry_of(a[0], GEMM, MXFP4);
    int leaf, k_first, extra;
    if (!e || !integer(a[5], &leaf) || !integer(a[6], &k_first) || !integer(a[8], &extra)) UNCOMMON;
    const int kind = e->kind;
    try {
        const at::Tensor *X = matrix(a[1], e->dtype), *W = matrix(a[3], e->dtype);
        if (!X || !W) UNCOMMON;
        const at::Tensor *Xs = nullptr, *Ws = nullptr;
        at::ScalarType out_type = at::kFloat;
        if (kind == GEMM || kind >= FP8) {                        // None there is for torch to answer: new_empty takes X's type
            if (!THPDtype_Check(a[7])) UNCOMMON;
            out_type = ((THPDtype *)a[7])->scalar_type;
        }
        if (type_code(out_type) < 0) UNCOMMON;
        const int M = (int)X->size(0);
        int K = (int)X->size(1), N;
        if (kind <= SWIGLU) {                                     // W [K, N]
            if (W->size(0) != K) UNCOMMON;
            N = (int)W->size(1);
            if (kind == SWIGLU) {
                if (N % 2) UNCOMMON;
                N /= 2;
            }
        } else {                                                  // W [N, bytes of K]
            if (W->size(1) != K) UNCOMMON;
            N = (int)W->size(0);
            if (kind != FP8) {
                Xs = matrix(a[2], at::kByte);
                Ws = matrix(a[4], at::kByte);
                if (!Xs || !Ws) UNCOMMON;
                if (kind == MXFP4) {
                    if (K > INT_MAX / 2) UNCOMMON;
                    K *= 2;
                } else if (extra >= 6) {                          // 6-bit elements: four in three bytes
                    if (K > INT_MAX / 4 || K % 3) UNCOMMON;
                    K = K / 3 * 4;
                }
                if (Xs->size(0) != M || Xs->size(1) != K / 32 || Ws->size(0) != N || Ws->size(1) != K / 32) UNCOMMON;
            }
        }
        const bool partials = kind == PARTIALS || kind == PARTIALS_F32;
        if (partials && extra < 1) UNCOMMON;
        at::Tensor Y = partials ? output({extra, M, N}, *X, at::kFloat)
                                : output({M, N}, *X, kind == SWIGLU ? e->dtype : kind == GEMM_F32 ? at::kFloat : out_type);
        if (!Y.defined()) UNCOMMON;
        void *stream = current_stream();
        Room ws;
        if (!room_for(e->need ? NEED(tbik_gemm_16bit_workspace_bytes)(M, N, K, leaf, k_first) : 0, a[1], *X, stream, &ws)) return nullptr;
        P x = X->data_ptr(), w = W->data_ptr(), y = Y.data_ptr(), xs = Xs ? Xs->data_ptr() : nullptr, wsc = Ws ? Ws->data_ptr() : nullptr;
        const L ldx = X->stride(0), ldw = W->stride(0), ldxs = Xs ? Xs->stride(0) : 0, ldws = Ws ? Ws->stride(0) : 0, ldy = partials ? 0 : Y.stride(0);
        const tbik_dtype yt = (tbik_dtype)type_code(Y.scalar_type());
        int st = 0;
        Py_BEGIN_ALLOW_THREADS
        switch (kind) {
            case GEMM:
            case SWIGLU: st = CALL(tbik_gemm)(x, ldx, w, ldw, y, ldy, yt, M, N, K, leaf, k_first, ws.at, ws.bytes, stream); break;
            case GEMM_F32: st = CALL(tbik_gemm_f32)(x, ldx, w, ldw, y, ldy, M, N, K, leaf, k_first, ws.at, ws.bytes, stream); break;
            case PARTIALS:
            case PARTIALS_F32: st = CALL(tbik_gemm_shard_partials)(x, ldx, w, ldw, (float *)y, M, N, K, leaf, k_first, extra, ws.at, ws.bytes, stream); break;
            case FP8: st = CALL(tbik_gemm_fp8)(x, ldx, w, ldw, y, ldy, yt, (tbik_dtype)extra, M, N, K, leaf, k_first, ws.at, ws.bytes, stream); break;
            case MX: st = CALL(tbik_gemm_mxfp8)(x, ldx, xs, ldxs, w, ldw, wsc, ldws, y, ldy, yt, (tbik_dtype)extra, M, N, K, leaf, k_first, ws.at, ws.bytes, stream); break;
            case MXFP4: st = CALL(tbik_gemm_mxfp4)(x, ldx, xs, ldxs, w, ldw, wsc, ldws, y, ldy, yt, M, N, K, leaf, k_first, ws.at, ws.bytes, stream); break;
        }
        Py_END_ALLOW_THREADS
        return wrapped(std::move(Y), st);
    } catch (const std::exception &) {
        if (PyErr_Occurred()) return nullptr;
        UNCOMMON;
    }
}

// rmsnorm(entry, x, weight, eps)
PyObject *rmsnorm(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 4) UNCOMMON;
    const Entry *e = entry_of(a[0], RMSNORM, RMSNORM);
    float eps;
    if (!e || !number(a[3], &eps)) UNCOMMON;
    try {
        const at::Tensor *x = matrix(a[1], e->dtype), *w = plain(a[2], 1);
        if (!x || !w || !x->is_contiguous() || !w->is_contiguous() || w->scalar_type() != e->dtype || w->numel() != x->size(1)) UNCOMMON;
        at::Tensor y = output({x->size(0), x->size(1)}, *x, e->dtype);
        if (!y.defined()) UNCOMMON;
        P px = x->data_ptr(), pw = w->data_ptr(), py = y.data_ptr(), stream = current_stream();
        const int M = (int)x->size(0), H = (int)x->size(1);
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = CALL(tbik_rmsnorm)(px, pw, py, M, H, eps, stream);
        Py_END_ALLOW_THREADS
        return wrapped(std::move(y), st);
    } catch (const std::exception &) {
        if (PyErr_Occurred()) return nullptr;
        UNCOMMON;
    }
}

// combine(entry, partials, residual, weight, eps) -> (hidden, normed)
PyObject *combine(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 5) UNCOMMON;
    const Entry *e = entry_of(a[0], COMBINE, COMBINE);
    float eps;
    if (!e || !number(a[4], &eps)) UNCOMMON;
    try {
        const at::Tensor *p = plain(a[1], 3), *r = matrix(a[2], e->dtype), *w = plain(a[3], 1);
        if (!p || !r || !w || p->scalar_type() != at::kFloat || !p->is_contiguous() || !r->is_contiguous() || w->scalar_type() != e->dtype || !w->is_contiguous() ||
            p->size(0) > INT_MAX || r->size(0) != p->size(1) || r->size(1) != p->size(2) || w->size(0) != p->size(2))
            UNCOMMON;
        at::Tensor h = output({r->size(0), r->size(1)}, *r, e->dtype), y = output({r->size(0), r->size(1)}, *r, e->dtype);
        if (!h.defined() || !y.defined()) UNCOMMON;
        P pp = p->data_ptr(), pr = r->data_ptr(), pw = w->data_ptr(), ph = h.data_ptr(), py = y.data_ptr(), stream = current_stream();
        const int shards = (int)p->size(0), M = (int)r->size(0), H = (int)r->size(1);
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = CALL(tbik_combine_residual_rmsnorm)((const float *)pp, shards, pr, pw, eps, ph, py, M, H, stream);
        Py_END_ALLOW_THREADS
        if (st) return PyLong_FromLong(st);
        PyObject *hidden = THPVariable_Wrap(std::move(h));
        if (!hidden) return nullptr;
        PyObject *normed = THPVariable_Wrap(std::move(y));
        if (!normed) {
            Py_DECREF(hidden);
            return nullptr;
        }
        PyObject *both = PyTuple_Pack(2, hidden, normed);
        Py_DECREF(hidden);
        Py_DECREF(normed);
        return both;
    } catch (const std::exception &) {
        if (PyErr_Occurred()) return nullptr;
        UNCOMMON;
    }
}

// row_reduce(entry, x, op)
PyObject *row_reduce(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 3) UNCOMMON;
    const Entry *e = entry_of(a[0], ROWS, ROWS);
    int op;
    if (!e || !integer(a[2], &op)) UNCOMMON;
    try {
        const at::Tensor *x = plain(a[1], 2);
        if (!x || !x->is_contiguous() || type_code(x->scalar_type()) < 0 || x->size(0) > INT_MAX) UNCOMMON;
        const int M = (int)x->size(0);
        const L V = x->size(1);
        at::Tensor y = op == TBIK_LOGSOFTMAX ? output({M, V}, *x, at::kFloat) : output({M}, *x, at::kFloat);
        if (!y.defined()) UNCOMMON;
        void *stream = current_stream();
        Room ws;
        // (the binding always passes a workspace here, of 256 bytes at least)
        const size_t need = NEED(tbik_row_reduce_workspace_bytes)(M, V, (tbik_rowop)op);
        if (!room_for(need ? need : 1, a[1], *x, stream, &ws)) return nullptr;
        P px = x->data_ptr(), py = y.data_ptr();
        const tbik_dtype t = (tbik_dtype)type_code(x->scalar_type());
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = CALL(tbik_row_reduce)(px, t, py, (tbik_rowop)op, M, V, ws.at, ws.bytes, stream);
        Py_END_ALLOW_THREADS
        return wrapped(std::move(y), st);
    } catch (const std::exception &) {
        if (PyErr_Occurred()) return nullptr;
        UNCOMMON;
    }
}

// attention(entry, Q, K, V, cu_q, cu_k, max_seqlen_q, scale, causal, max_seqlen_k)
PyObject *attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 10) UNCOMMON;
    const Entry *e = entry_of(a[0], ATTENTION, ATTENTION);
    int max_q, max_k;
    float scale;
    if (!e || !integer(a[6], &max_q) || !number(a[7], &scale) || !PyBool_Check(a[8]) || !integer(a[9], &max_k)) UNCOMMON;
    try {
        const at::Tensor *t[3];
        for (int i = 0; i < 3; ++i) {
            t[i] = plain(a[1 + i], 3);
            if (!t[i] || t[i]->scalar_type() != e->dtype || t[i]->stride(2) != 1 || t[i]->stride(1) != t[i]->size(2) || t[i]->size(0) > INT_MAX || t[i]->size(1) > INT_MAX) UNCOMMON;
        }
        const at::Tensor &Q = *t[0], &K = *t[1], &V = *t[2];
        const at::Tensor *cq = plain(a[4], 1), *ck = plain(a[5], 1);
        if (!cq || !ck || cq->scalar_type() != at::kInt || ck->scalar_type() != at::kInt || !cq->is_contiguous() || !ck->is_contiguous() || cq->numel() < 1 ||
            cq->numel() != ck->numel() || cq->numel() > INT_MAX || K.size(0) != V.size(0) || K.size(1) != V.size(1) || K.size(2) != V.size(2) || K.size(2) != Q.size(2) ||
            Q.size(2) != 128)
            UNCOMMON;
        const int batch = (int)cq->numel() - 1, Tq = (int)Q.size(0), Tk = (int)K.size(0), Hq = (int)Q.size(1), Hkv = (int)K.size(1);
        at::Tensor O = output({Tq, Hq, 128}, Q, e->dtype);
        if (!O.defined()) UNCOMMON;
        void *stream = current_stream();
        Room ws;
        if (!room_for(NEED(tbik_attention_workspace_bytes)(batch, max_q, max_k < Tk ? max_k : Tk, Hq, Hkv), a[1], Q, stream, &ws)) return nullptr;
        P q = Q.data_ptr(), k = K.data_ptr(), v = V.data_ptr(), o = O.data_ptr(), pq = cq->data_ptr(), pk = ck->data_ptr();
        const L sq = Q.stride(0), sk = K.stride(0), sv = V.stride(0), so = O.stride(0);
        const int causal = a[8] == Py_True;
        int st;
        Py_BEGIN_ALLOW_THREADS
        st = CALL(tbik_attention)(
            q, k, v, o, (const int32_t *)pq, (const int32_t *)pk, batch, max_q, max_k, Tq, Tk, Hq, Hkv, 128, sq, sk, sv, so, scale, causal, ws.at, ws.bytes, stream);
        Py_END_ALLOW_THREADS
        return wrapped(std::move(O), st);
    } catch (const std::exception &) {
        if (PyErr_Occurred()) return nullptr;
        UNCOMMON;
    }
}

// register(entry, kind, address, address of the workspace query or 0, operand dtype)
PyObject *register_entry(PyObject *, PyObject *args) {
    int i, kind;
    unsigned long long call, need;
    PyObject *dtype;
    if (!PyArg_ParseTuple(args, "iiKKO", &i, &kind, &call, &need, &dtype)) return nullptr;
    if (i < 0 || i >= MAX_ENTRIES || kind < 0 || kind >= KINDS || !call || !THPDtype_Check(dtype)) {
        PyErr_SetString(PyExc_ValueError, "entry");
        return nullptr;
    }
    entries[i].kind = kind;
    entries[i].call = (void *)(uintptr_t)call;
    entries[i].need = (void *)(uintptr_t)need;
    entries[i].dtype = ((THPDtype *)dtype)->scalar_type;
    Py_RETURN_NONE;
}

// use(dict of workspaces, function that makes one)
PyObject *use(PyObject *, PyObject *args) {
    PyObject *d, *f;
    if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &d, &f)) return nullptr;
    Py_INCREF(d);
    Py_INCREF(f);
    Py_XDECREF(workspaces);
    Py_XDECREF(make_workspace);
    workspaces = d;
    make_workspace = f;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"product", (PyCFunction)(void (*)(void))product, METH_FASTCALL, nullptr},
    {"rmsnorm", (PyCFunction)(void (*)(void))rmsnorm, METH_FASTCALL, nullptr},
    {"combine", (PyCFunction)(void (*)(void))combine, METH_FASTCALL, nullptr},
    {"row_reduce", (PyCFunction)(void (*)(void))row_reduce, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void (*)(void))attention, METH_FASTCALL, nullptr},
    {"register", register_entry, METH_VARARGS, nullptr},
    {"use", use, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
