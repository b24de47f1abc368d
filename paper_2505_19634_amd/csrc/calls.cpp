// The host side of the calls that are shorter on the GPU than in Python: argument checks, the descriptor and the library call of
// verify_attention (and its _noalloc form), spec_accept, majority_vote and skinny_gemm, as a CPython extension on torch's tensors.  binding.py keeps
// the signatures, makes what a caller leaves out and holds the workspaces; a call that finds its workspace missing or too small
// says how much it needs and is made again.
// Measured (2 branches, fp32, vocabulary 1000): a step's three calls through ctypes are 6.5 + 6.5 + 4.1 us of host time for
// three launches of 2.7 us each, and their kernels take 11 us together; through here 4.1 + 4.0 + 3.4 us, the step 16.7 -> 12.7.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "lotts.h"

namespace {

// entry points of the liblotts build in use, bound by address: the extension itself links against none
using attn_ws_fn = decltype(&verify_attention_workspace_bytes);
using attn_fn = decltype(&verify_attention);
using attn_noalloc_fn = decltype(&verify_attention_noalloc);
using accept_ws_fn = decltype(&spec_accept_workspace_bytes);
using accept_fn = decltype(&spec_accept);
using vote_fn = decltype(&majority_vote);
using gemm_ws_fn = decltype(&skinny_gemm_workspace_bytes);
using gemm_fn = decltype(&skinny_gemm);

struct Calls {
    PyObject_HEAD
    attn_ws_fn attn_ws;
    attn_fn attn;
    accept_ws_fn accept_ws;
    accept_fn accept;
    vote_fn vote;
    gemm_ws_fn gemm_ws;
    gemm_fn gemm;
    attn_noalloc_fn attn_noalloc;
};

struct Error {  // a Python exception to raise
    PyObject* type;
    const char* text;
};

const at::Tensor& tensor(PyObject* o, const char* what) {
    if (!THPVariable_Check(o)) throw Error{PyExc_TypeError, what};
    return THPVariable_Unpack(o);
}
bool is(const at::Tensor& t, at::ScalarType type) { return t.scalar_type() == type && t.is_contiguous(); }

// The workspace of a call: the caller's as it is, or the cached one if it is large enough; false if that is not there.
bool workspace(PyObject* own, PyObject* cached, size_t need, void** ptr, size_t* bytes) {
    PyObject* o = own != Py_None ? own : cached;
    if (o == Py_None) return false;
    const at::Tensor& t = tensor(o, "the workspace must be a tensor");
    *ptr = t.data_ptr();
    *bytes = t.nbytes();
    return own != Py_None || *bytes >= need;
}

// Status of a call, 0 or negative; a positive number asks for that many bytes of workspace.
template <typename F>
PyObject* guarded(F body) {
    try {
        return PyLong_FromSsize_t(body());
    } catch (const Error& e) {
        PyErr_SetString(e.type, e.text);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}
template <typename F>
Py_ssize_t released(F call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return rc;
}
void* address(PyObject* o) { return PyLong_AsVoidPtr(o); }
void expect(Py_ssize_t n, Py_ssize_t want) {
    if (n != want) throw Error{PyExc_TypeError, "wrong number of arguments"};
}
constexpr Py_ssize_t kNoWorkspaceQuery = -2;  // a size of 0: the geometry cannot be served

// At least as large in every dimension: what a kernel addresses by the other tensor's sizes lies inside this one.
bool covers(const at::Tensor& t, at::IntArrayRef wanted) {
    const at::IntArrayRef sizes = t.sizes();
    if (sizes.size() != wanted.size()) return false;
    for (size_t i = 0; i < sizes.size(); ++i)
        if (sizes[i] < wanted[i]) return false;
    return true;
}
bool expanded(const at::Tensor& t) {
    const at::IntArrayRef sizes = t.sizes(), strides = t.strides();
    for (size_t i = 0; i < sizes.size(); ++i)
        if (strides[i] == 0 && sizes[i] > 1) return true;
    return false;
}
// One of the outputs with a number for each row: dense and long enough.
template <typename T>
T* rows_of(PyObject* o, at::ScalarType type, int64_t rows, const char* what) {
    const at::Tensor& t = tensor(o, what);
    if (!is(t, type)) throw Error{PyExc_TypeError, what};
    if (t.numel() < rows) throw Error{PyExc_ValueError, what};
    return static_cast<T*>(t.data_ptr());
}

struct Attention {  // the descriptor and the pointers of a call
    lotts_attn_desc d = {};
    const void *q, *kpre = nullptr, *vpre = nullptr, *kpriv, *vpriv;
    const int32_t* len;
    void* out;
    float* lse = nullptr;
};
// a: Q, Kpre, Vpre, Kpriv, Vpriv, priv_len, scale, out, lse.  Whatever the kernels address lies inside the tensors: they know pointers and
// strides alone, and a stride of 0 means the dense layout to them.
Attention attention(PyObject* const* a) {
    const at::Tensor &Q = tensor(a[0], "Q must be a tensor"), &Kpriv = tensor(a[3], "Kpriv must be a tensor"),
                     &Vpriv = tensor(a[4], "Vpriv must be a tensor"), &len = tensor(a[5], "priv_len must be a tensor"),
                     &O = tensor(a[7], "out must be a tensor");
    const at::Tensor *Kpre = nullptr, *Vpre = nullptr;
    if (a[1] != Py_None) {
        Kpre = &tensor(a[1], "Kpre must be a tensor");
        if (Kpre->dim() != 3) throw Error{PyExc_ValueError, "Kpre must be [Hkv][P][D]"};
        if (Kpre->size(1) == 0) Kpre = nullptr;
        else Vpre = &tensor(a[2], "Vpre must be a tensor");
    }
    if (Q.dim() != 4 || Kpriv.dim() != 4 || O.dim() != 4) throw Error{PyExc_ValueError, "Q and out must be [B][k+1][Hq][D], Kpriv [B][Hkv][Lmax][D]"};
    if (Vpriv.strides() != Kpriv.strides() || (Kpre && Vpre->strides() != Kpre->strides()))
        throw Error{PyExc_ValueError, "K and V of a segment must share strides"};
    if (len.scalar_type() != at::kInt) throw Error{PyExc_TypeError, "priv_len must be int32"};
    if (Kpriv.sizes()[0] != Q.sizes()[0] || Kpriv.sizes()[3] != Q.sizes()[3]) throw Error{PyExc_ValueError, "Q and Kpriv disagree"};
    Attention c;
    lotts_attn_desc& d = c.d;
    if (Q.scalar_type() == at::kBFloat16) d.dtype = LOTTS_BF16;
    else if (Q.scalar_type() == at::kFloat) d.dtype = LOTTS_F32;
    else throw Error{PyExc_TypeError, "Q/K/V must be bfloat16 or float32"};
    const at::ScalarType type = Q.scalar_type();
    for (const at::Tensor* t : {&Q, &Kpriv, &O, Kpre}) {
        if (!t) continue;
        if (t->strides().back() != 1) throw Error{PyExc_ValueError, "the head dimension must be contiguous"};
        if (expanded(*t)) throw Error{PyExc_ValueError, "expanded tensors are not supported"};
    }
    for (const at::Tensor* t : {&Kpriv, &Vpriv, &O, Kpre, Vpre})
        if (t && t->scalar_type() != type) throw Error{PyExc_TypeError, "Q, K, V and out share one dtype"};
    const at::IntArrayRef q = Q.sizes(), own = Kpriv.sizes();
    if (!covers(O, q)) throw Error{PyExc_ValueError, "out must be [B][k+1][Hq][D]"};
    if (!covers(Vpriv, own)) throw Error{PyExc_ValueError, "Vpriv must be [B][Hkv][Lmax][D]"};
    if (Kpre) {
        const int64_t prefix[] = {own[1], Kpre->sizes()[1], q[3]};
        if (!covers(*Kpre, prefix) || !covers(*Vpre, prefix)) throw Error{PyExc_ValueError, "Kpre and Vpre must be [Hkv][P][D]"};
    }
    if (!len.is_contiguous() || len.numel() < q[0]) throw Error{PyExc_ValueError, "priv_len must be contiguous [B]"};
    d.B = (int32_t)q[0];
    d.k = (int32_t)q[1] - 1;
    d.Hq = (int32_t)q[2];
    d.D = (int32_t)q[3];
    d.Hkv = (int32_t)own[1];
    d.Lmax = (int32_t)own[2];
    d.scale = (float)PyFloat_AsDouble(a[6]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw Error{PyExc_TypeError, "scale must be a number"};
    }
    const at::IntArrayRef qs = Q.strides(), os = O.strides(), ks = Kpriv.strides();
    d.q_stride_b = qs[0], d.q_stride_r = qs[1], d.q_stride_h = qs[2];
    d.o_stride_b = os[0], d.o_stride_r = os[1], d.o_stride_h = os[2];
    d.kpriv_stride_b = ks[0], d.kpriv_stride_h = ks[1], d.kpriv_stride_t = ks[2];
    c.q = Q.data_ptr(), c.kpriv = Kpriv.data_ptr(), c.vpriv = Vpriv.data_ptr(), c.out = O.data_ptr();
    c.len = static_cast<const int32_t*>(len.data_ptr());
    if (Kpre) {
        d.P = (int32_t)Kpre->sizes()[1];
        d.kpre_stride_h = Kpre->strides()[0], d.kpre_stride_t = Kpre->strides()[1];
        c.kpre = Kpre->data_ptr(), c.vpre = Vpre->data_ptr();
    }
    if (a[8] != Py_None) c.lse = rows_of<float>(a[8], at::kFloat, q[0] * q[1] * q[2], "lse must be contiguous float32 [B][k+1][Hq]");
    return c;
}

// Q, Kpre, Vpre, Kpriv, Vpriv, priv_len, scale, out, lse, workspace, cached workspace, stream
PyObject* call_attention(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Calls* c = reinterpret_cast<Calls*>(self);
    return guarded([&]() -> Py_ssize_t {
        expect(n, 12);
        const Attention t = attention(a);
        const size_t need = c->attn_ws(&t.d);
        if (need == 0) return kNoWorkspaceQuery;
        void* ws;
        size_t bytes;
        if (!workspace(a[9], a[10], need, &ws, &bytes)) return (Py_ssize_t)need;
        void* stream = address(a[11]);
        return released([&] { return c->attn(&t.d, t.q, t.kpre, t.vpre, t.kpriv, t.vpriv, t.len, t.out, t.lse, ws, bytes, stream); });
    });
}

// Q, Kpre, Vpre, Kpriv, Vpriv, priv_len, scale, out, lse, stream
PyObject* call_attention_noalloc(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Calls* c = reinterpret_cast<Calls*>(self);
    return guarded([&]() -> Py_ssize_t {
        expect(n, 10);
        const Attention t = attention(a);
        void* stream = address(a[9]);
        return released([&] { return c->attn_noalloc(&t.d, t.q, t.kpre, t.vpre, t.kpriv, t.vpriv, t.len, t.out, t.lse, stream); });
    });
}

// p, q, draft, u, accept_len, next_token, workspace, cached workspace, stream
PyObject* call_accept(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Calls* c = reinterpret_cast<Calls*>(self);
    return guarded([&]() -> Py_ssize_t {
        expect(n, 9);
        const at::Tensor &p = tensor(a[0], "p must be a tensor"), &u = tensor(a[3], "u must be a tensor");
        if (p.dim() != 3) throw Error{PyExc_ValueError, "p must be [B][k+1][V]"};
        const int64_t B = p.size(0), R = p.size(1), V = p.size(2), k = R - 1;
        if (!is(p, at::kFloat) || !is(u, at::kFloat)) throw Error{PyExc_TypeError, "p and u must be contiguous float32"};
        if (u.dim() != 2 || u.size(0) != B || u.size(1) != R) throw Error{PyExc_ValueError, "u must be [B][k+1]"};
        const float* q = nullptr;
        const int32_t* draft = nullptr;
        if (k > 0) {
            if (a[1] == Py_None || a[2] == Py_None) throw Error{PyExc_ValueError, "q must be [B][k][V] and draft [B][k]"};
            const at::Tensor &tq = tensor(a[1], "q must be a tensor"), &td = tensor(a[2], "draft must be a tensor");
            if (tq.dim() != 3 || tq.size(0) != B || tq.size(1) != k || tq.size(2) != V || td.dim() != 2 || td.size(0) != B || td.size(1) != k)
                throw Error{PyExc_ValueError, "q must be [B][k][V] and draft [B][k]"};
            if (!is(tq, at::kFloat) || !is(td, at::kInt)) throw Error{PyExc_TypeError, "q must be contiguous float32 and draft contiguous int32"};
            q = static_cast<const float*>(tq.data_ptr());
            draft = static_cast<const int32_t*>(td.data_ptr());
        }
        const size_t need = c->accept_ws((int32_t)B, (int32_t)k, (int32_t)V);
        if (need == 0) return kNoWorkspaceQuery;
        void* ws;
        size_t bytes;
        if (!workspace(a[6], a[7], need, &ws, &bytes)) return (Py_ssize_t)need;
        const float *pp = static_cast<const float*>(p.data_ptr()), *up = static_cast<const float*>(u.data_ptr());
        int32_t* len = rows_of<int32_t>(a[4], at::kInt, B, "accept_len must be contiguous int32 [B]");
        int32_t* next = rows_of<int32_t>(a[5], at::kInt, B, "next_token must be contiguous int32 [B]");
        void* stream = address(a[8]);
        return released([&] { return c->accept((int32_t)B, (int32_t)k, (int32_t)V, pp, q, draft, up, len, next, ws, bytes, stream); });
    });
}

// answers [N][B], winner, winner_count, stream
PyObject* call_vote(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Calls* c = reinterpret_cast<Calls*>(self);
    return guarded([&]() -> Py_ssize_t {
        expect(n, 4);
        const at::Tensor& answers = tensor(a[0], "answers must be a tensor");
        if (!is(answers, at::kInt)) throw Error{PyExc_TypeError, "answers must be contiguous int32"};
        if (answers.dim() != 2) throw Error{PyExc_ValueError, "answers must be [N][B]"};
        const int32_t N = (int32_t)answers.size(0), B = (int32_t)answers.size(1);
        const int32_t* src = static_cast<const int32_t*>(answers.data_ptr());
        int32_t* winner = rows_of<int32_t>(a[1], at::kInt, N, "winner must be contiguous int32 [N]");
        int32_t* count = rows_of<int32_t>(a[2], at::kInt, N, "winner_count must be contiguous int32 [N]");
        void* stream = address(a[3]);
        return released([&] { return c->vote(N, B, src, winner, count, stream); });
    });
}

// X, W, out, workspace, cached workspace, stream
PyObject* call_gemm(PyObject* self, PyObject* const* a, Py_ssize_t n) {
    const Calls* c = reinterpret_cast<Calls*>(self);
    return guarded([&]() -> Py_ssize_t {
        expect(n, 6);
        const at::Tensor &X = tensor(a[0], "X must be a tensor"), &W = tensor(a[1], "W must be a tensor"), &Y = tensor(a[2], "out must be a tensor");
        if (X.dim() != 2 || W.dim() != 2 || W.size(1) != X.size(1) || X.stride(1) != 1 || W.stride(1) != 1)
            throw Error{PyExc_ValueError, "X [M][K] and W [N][K] must share K and have contiguous rows"};
        const int64_t shape[] = {X.size(0), W.size(0)};
        if (Y.scalar_type() != at::kBFloat16) throw Error{PyExc_TypeError, "out must be bfloat16"};
        int64_t row = 1;  // elements of a row of out that lie next to each other
        for (int64_t i = Y.dim() - 1; i > 0 && (Y.size(i) == 1 || Y.stride(i) == row); --i) row *= Y.size(i);
        if (Y.dim() < 2 || Y.size(0) < shape[0] || row < shape[1]) throw Error{PyExc_ValueError, "out must be [M][N] with contiguous rows"};
        const int32_t M = (int32_t)X.size(0), N = (int32_t)W.size(0), K = (int32_t)X.size(1);
        const size_t need = c->gemm_ws(M, N, K);
        if (need == 0) return kNoWorkspaceQuery;
        void* ws;
        size_t bytes;
        if (!workspace(a[3], a[4], need, &ws, &bytes)) return (Py_ssize_t)need;
        const void *x = X.data_ptr(), *w = W.data_ptr();
        void* y = Y.data_ptr();
        const int64_t ldx = X.stride(0), ldw = W.stride(0), ldy = Y.stride(0);
        void* stream = address(a[5]);
        return released([&] { return c->gemm(M, N, K, x, ldx, w, ldw, y, ldy, ws, bytes, stream); });
    });
}

// Calls(address of verify_attention_workspace_bytes, verify_attention, spec_accept_workspace_bytes, spec_accept, majority_vote,
// skinny_gemm_workspace_bytes, skinny_gemm, verify_attention_noalloc)
PyObject* calls_new(PyTypeObject* type, PyObject* args, PyObject*) {
    void* f[8];
    if (PyTuple_GET_SIZE(args) != 8) {
        PyErr_SetString(PyExc_TypeError, "eight addresses");
        return nullptr;
    }
    for (int i = 0; i < 8; ++i) {
        f[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(args, i));
        if (!f[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an address is 0");
            return nullptr;
        }
    }
    Calls* c = reinterpret_cast<Calls*>(type->tp_alloc(type, 0));
    if (!c) return nullptr;
    c->attn_ws = reinterpret_cast<attn_ws_fn>(f[0]);
    c->attn = reinterpret_cast<attn_fn>(f[1]);
    c->accept_ws = reinterpret_cast<accept_ws_fn>(f[2]);
    c->accept = reinterpret_cast<accept_fn>(f[3]);
    c->vote = reinterpret_cast<vote_fn>(f[4]);
    c->gemm_ws = reinterpret_cast<gemm_ws_fn>(f[5]);
    c->gemm = reinterpret_cast<gemm_fn>(f[6]);
    c->attn_noalloc = reinterpret_cast<attn_noalloc_fn>(f[7]);
    return reinterpret_cast<PyObject*>(c);
}

PyMethodDef calls_methods[] = {
    {"verify_attention", (PyCFunction)(void (*)(void))call_attention, METH_FASTCALL, nullptr},
    {"verify_attention_noalloc", (PyCFunction)(void (*)(void))call_attention_noalloc, METH_FASTCALL, nullptr},
    {"spec_accept", (PyCFunction)(void (*)(void))call_accept, METH_FASTCALL, nullptr},
    {"majority_vote", (PyCFunction)(void (*)(void))call_vote, METH_FASTCALL, nullptr},
    {"skinny_gemm", (PyCFunction)(void (*)(void))call_gemm, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef calls_module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
    calls_type.tp_name = "_calls.Calls";
    calls_type.tp_basicsize = sizeof(Calls);
    calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
    calls_type.tp_new = calls_new;
    calls_type.tp_methods = calls_methods;
    if (PyType_Ready(&calls_type) < 0) return nullptr;
    PyObject* m = PyModule_Create(&calls_module);
    if (!m) return nullptr;
    Py_INCREF(&calls_type);
    if (PyModule_AddObject(m, "Calls", reinterpret_cast<PyObject*>(&calls_type)) < 0) {
        Py_DECREF(&calls_type);
        Py_DECREF(m);
        return nullptr;
    }
    if (PyModule_AddStringConstant(m, "built_for_torch", LOTTS_TORCH) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
