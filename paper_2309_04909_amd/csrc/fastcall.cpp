// Argument marshalling of the small calls in native code (Python extension
// module paper_2309_04909_amd._fastcall).
//
// A call on a few thousand elements is bound by the host: on MI355X's host
// the launch itself takes 2.5-3.8 us, and checking four tensors, taking their
// pointers and converting eleven ctypes arguments in Python added 2.4 us to
// it.  These functions do the same checks on the tensors directly and call
// the C ABI through its address.  They handle the plain case only: anything
// else (another type, a wrong size, an odd integer, no contiguous storage)
// returns None, and the Python binding takes the call from there, with its
// own checks and errors.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <string.h>

#include "../../include/bicop.h"

namespace {

PyObject* g_check = nullptr;      // bicop._check(rc, where): raises BicopError
PyObject* g_struct = nullptr;     // "_c"
PyObject* g_c = nullptr;          // "c"
PyObject* g_stream = nullptr;     // "cuda_stream"

// A copy of a Params / Seeds object's C structure (the ctypes object in its
// _c, which c() builds), or false with no error set.
template <typename S>
bool take_struct(PyObject* o, S* out) {
    PyObject* c = PyObject_GetAttr(o, g_struct);
    if (!c) {
        PyErr_Clear();
        c = PyObject_CallMethodNoArgs(o, g_c);
    }
    bool ok = false;
    Py_buffer v;
    if (c && PyObject_GetBuffer(c, &v, PyBUF_SIMPLE) == 0) {
        ok = v.len == (Py_ssize_t)sizeof(S);
        if (ok) memcpy(out, v.buf, sizeof(S));
        PyBuffer_Release(&v);
    }
    Py_XDECREF(c);
    if (!ok) PyErr_Clear();
    return ok;
}

bool as_u64(PyObject* o, uint64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsUnsignedLongLong(o);
    if (*v == (uint64_t)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool as_u32(PyObject* o, uint32_t* v) {
    uint64_t w;
    if (!as_u64(o, &w) || w > 0xFFFFFFFFull) return false;
    *v = (uint32_t)w;
    return true;
}

uint32_t width_of(uint32_t ell) { return ell <= 32 ? 4 : 8; }

const at::Tensor* plain_tensor(PyObject* o, uint32_t width) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.is_sparse() || t.element_size() != width || !t.is_contiguous()) return nullptr;
    return &t;
}

// The interpreter lock released for a scope, also when the scope is left by
// an exception: the C calls, as ctypes makes them, and the allocations, which
// can wait for the device.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// An owned reference to a call's result.
struct Result {
    PyObject* o = nullptr;
    ~Result() { Py_XDECREF(o); }
};

// The stream to enqueue on: `stream`, else the current one of t's device.
bool take_stream(PyObject* stream, const at::Tensor& t, void** out) {
    if (stream == Py_None) {
        *out = c10::hip::getCurrentHIPStream(t.get_device()).stream();
        return true;
    }
    PyObject* h = PyObject_GetAttr(stream, g_stream);
    uint64_t v = 0;
    const bool ok = h && as_u64(h, &v);
    Py_XDECREF(h);
    if (!ok) PyErr_Clear();
    *out = reinterpret_cast<void*>(v);
    return ok;
}

// One output of `like`'s device: the given tensor if it has n elements of
// `width` bytes, or a new one of `sizes` and type `dtype`.  The reference goes
// to *o, the pointer to *ptr.
bool take_output(PyObject* given, const at::Tensor& like, at::IntArrayRef sizes, at::ScalarType dtype, uint32_t width,
                 int64_t n, PyObject** o, void** ptr) {
    if (given == Py_None) {
        at::Tensor t;
        {
            Unlocked unlocked;
            t = at::empty(sizes, like.options().dtype(dtype).requires_grad(false));
        }
        *ptr = t.data_ptr();
        *o = THPVariable_Wrap(std::move(t));
        if (!*o) PyErr_Clear();
        return *o != nullptr;
    }
    const at::Tensor* t = plain_tensor(given, width);
    if (!t || t->numel() != n) return false;
    *ptr = t->data_ptr();
    Py_INCREF(given);
    *o = given;
    return true;
}

at::ScalarType ring_type(uint32_t width) { return width == 4 ? at::kUInt32 : at::kUInt64; }

// K share arrays of one length (x[0..K)), their K outputs (a tuple, or new ones
// shaped like the inputs; the result) and the stream of one call.
template <int K>
struct Shares {
    void *x[K], *y[K];
    uint64_t n;
    void* stream;
    Result result;

    bool take(PyObject* const* in, uint32_t win, uint32_t wout, PyObject* out, PyObject* ostream) {
        const at::Tensor* t[K];
        for (int k = 0; k < K; ++k) {
            t[k] = plain_tensor(in[k], win);
            if (!t[k] || t[k]->numel() != t[0]->numel()) return false;
            x[k] = t[k]->data_ptr();
        }
        n = (uint64_t)t[0]->numel();
        if (!take_stream(ostream, *t[0], &stream)) return false;
        if (out != Py_None && (!PyTuple_CheckExact(out) || PyTuple_GET_SIZE(out) != K)) return false;
        PyObject* r = PyTuple_New(K);
        if (!r) {
            PyErr_Clear();
            return false;
        }
        result.o = r;
        for (int k = 0; k < K; ++k) {
            PyObject* o = nullptr;
            if (!take_output(out == Py_None ? Py_None : PyTuple_GET_ITEM(out, k), *t[k], t[k]->sizes(), ring_type(wout), wout,
                             (int64_t)n, &o, &y[k]))
                return false;
            PyTuple_SET_ITEM(r, k, o);
        }
        return true;
    }
};

// Ends a call: its result, or the binding's exception for rc != 0.
PyObject* conclude(Result& result, int rc, PyObject* name) {
    if (rc == 0) {
        PyObject* o = result.o;
        result.o = nullptr;
        return o;
    }
    PyObject* code = PyLong_FromLong(rc);
    PyObject* r = code ? PyObject_CallFunctionObjArgs(g_check, code, name, nullptr) : nullptr;
    Py_XDECREF(code);
    Py_XDECREF(r);
    if (r) PyErr_SetString(PyExc_RuntimeError, "the library refused the call");
    return nullptr;
}

// fn(args) without the GIL, as ctypes calls it.
template <typename Fn>
int unlocked(Fn&& fn) {
    Unlocked u;
    return fn();
}

using DreluFn = int (*)(const void*, const void*, void*, void*, uint64_t, const bc_drelu_params*, const bc_seeds*, uint64_t,
                        void*, bc_msg_acct*, void*);
using TruncFn = int (*)(const void*, const void*, void*, void*, uint64_t, uint32_t, uint32_t, const bc_drelu_params*,
                        const bc_seeds*, uint64_t, void*, bc_msg_acct*, void*);
using CutFn = int (*)(const void*, const void*, void*, void*, uint64_t, uint32_t, uint32_t, uint32_t, void*);

using RssFn = int (*)(const void*, const void*, const void*, void*, void*, void*, uint64_t, const bc_drelu_params*,
                      const bc_rss_seeds*, uint64_t, void*, bc_msg_acct*, void*);
using MulFn = int (*)(const void*, const void*, const void*, const void*, void*, void*, uint64_t, uint32_t, uint32_t, uint32_t,
                      const bc_seeds*, uint64_t, void*);
using SendFn = int (*)(uint32_t, const void*, uint32_t*, uint64_t, const bc_drelu_params*, const bc_seeds*, uint64_t, void*);
using ReplyFn = int (*)(const uint32_t*, const uint32_t*, void*, void*, uint64_t, const bc_drelu_params*, const bc_seeds*,
                        uint64_t, void*);
using FinishFn = int (*)(uint32_t, const void*, void*, uint64_t, const bc_drelu_params*, const bc_seeds*, uint64_t, void*);

// 32-bit words of one element's packed message (bc_msg_words), 0 for a window
// the library refuses.
int64_t words_of(const bc_drelu_params& prm) {
    const int64_t np = (int64_t)prm.lx + 1;
    return np >= 2 && np <= 33 ? (np * np + 31) / 32 : 0;
}

// Each function's arguments: the C function's address, the binding's name of
// the call, then the binding's own arguments.  A function that throws (a
// tensor without storage, no memory) has enqueued nothing: None, and the
// binding's own path takes the call.
template <typename Body>
PyObject* guarded(Body&& body) {
    try {
        return body();
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// drelu(fn, name, x0, x1, params, seeds, elem_base, out, stream)
PyObject* py_drelu(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn, base;
        bc_drelu_params prm;
        bc_seeds seeds;
        if (nargs != 9 || !as_u64(a[0], &fn) || !as_u64(a[6], &base) || !take_struct(a[4], &prm) || !take_struct(a[5], &seeds))
            Py_RETURN_NONE;
        Shares<2> s;
        const uint32_t w = width_of(prm.ell);
        if (!s.take(a + 2, w, w, a[7], a[8])) Py_RETURN_NONE;
        return conclude(s.result, unlocked([&] {
            return reinterpret_cast<DreluFn>(fn)(s.x[0], s.x[1], s.y[0], s.y[1], s.n, &prm, &seeds, base, nullptr, nullptr,
                                                 s.stream);
        }), a[1]);
    });
}

// trunc(fn, name, x0, x1, ell_in, k1, params, seeds, elem_base, out, stream)
PyObject* py_trunc(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn, base;
        uint32_t ell_in, k1;
        bc_drelu_params prm;
        bc_seeds seeds;
        if (nargs != 11 || !as_u64(a[0], &fn) || !as_u32(a[4], &ell_in) || !as_u32(a[5], &k1) || !as_u64(a[8], &base) ||
            !take_struct(a[6], &prm) || !take_struct(a[7], &seeds))
            Py_RETURN_NONE;
        Shares<2> s;
        if (!s.take(a + 2, width_of(ell_in), width_of(prm.ell), a[9], a[10])) Py_RETURN_NONE;
        return conclude(s.result, unlocked([&] {
            return reinterpret_cast<TruncFn>(fn)(s.x[0], s.x[1], s.y[0], s.y[1], s.n, ell_in, k1, &prm, &seeds, base, nullptr,
                                                 nullptr, s.stream);
        }), a[1]);
    });
}

// cut(fn, name, x0, x1, ell, k1, k2, out, stream): bc_trunc_det
PyObject* py_cut(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn;
        uint32_t ell, k1, k2;
        if (nargs != 9 || !as_u64(a[0], &fn) || !as_u32(a[4], &ell) || !as_u32(a[5], &k1) || !as_u32(a[6], &k2) ||
            (uint64_t)k1 + k2 > ell)
            Py_RETURN_NONE;
        Shares<2> s;
        if (!s.take(a + 2, width_of(ell), width_of(ell - k1 - k2), a[7], a[8])) Py_RETURN_NONE;
        return conclude(s.result, unlocked([&] {
            return reinterpret_cast<CutFn>(fn)(s.x[0], s.x[1], s.y[0], s.y[1], s.n, ell, k1, k2, s.stream);
        }), a[1]);
    });
}

// rss(fn, name, (x0, x1, x2), params, seeds, elem_base, out, stream)
PyObject* py_rss(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn, base;
        bc_drelu_params prm;
        bc_rss_seeds seeds;
        if (nargs != 8 || !as_u64(a[0], &fn) || !PyTuple_CheckExact(a[2]) || PyTuple_GET_SIZE(a[2]) != 3 ||
            !as_u64(a[5], &base) || !take_struct(a[3], &prm) || !take_struct(a[4], &seeds))
            Py_RETURN_NONE;
        PyObject* in[3] = {PyTuple_GET_ITEM(a[2], 0), PyTuple_GET_ITEM(a[2], 1), PyTuple_GET_ITEM(a[2], 2)};
        Shares<3> s;
        const uint32_t w = width_of(prm.ell);
        if (!s.take(in, w, w, a[6], a[7])) Py_RETURN_NONE;
        return conclude(s.result, unlocked([&] {
            return reinterpret_cast<RssFn>(fn)(s.x[0], s.x[1], s.x[2], s.y[0], s.y[1], s.y[2], s.n, &prm, &seeds, base, nullptr,
                                               nullptr, s.stream);
        }), a[1]);
    });
}

// mul(fn, name, x0, x1, y0, y1, ell, f, order, seeds, elem_base, out, stream)
PyObject* py_mul(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn, base;
        uint32_t ell, f, order;
        bc_seeds seeds;
        if (nargs != 13 || !as_u64(a[0], &fn) || !as_u32(a[6], &ell) || !as_u32(a[7], &f) || !as_u32(a[8], &order) ||
            !as_u64(a[10], &base) || !take_struct(a[9], &seeds))
            Py_RETURN_NONE;
        const uint32_t w = width_of(ell);
        Shares<2> s;
        const at::Tensor *y0 = plain_tensor(a[4], w), *y1 = plain_tensor(a[5], w);
        if (!y0 || !y1 || !s.take(a + 2, w, w, a[11], a[12]) || (uint64_t)y0->numel() != s.n || (uint64_t)y1->numel() != s.n)
            Py_RETURN_NONE;
        const void *p0 = y0->data_ptr(), *p1 = y1->data_ptr();
        return conclude(s.result, unlocked([&] {
            return reinterpret_cast<MulFn>(fn)(s.x[0], s.x[1], p0, p1, s.y[0], s.y[1], s.n, ell, f, order, &seeds, base, s.stream);
        }), a[1]);
    });
}

// send(fn, name, party, x, params, seeds, elem_base, out, stream)
PyObject* py_send(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn, base;
        uint32_t party;
        bc_drelu_params prm;
        bc_seeds seeds;
        if (nargs != 9 || !as_u64(a[0], &fn) || !as_u32(a[2], &party) || !as_u64(a[6], &base) || !take_struct(a[4], &prm) ||
            !take_struct(a[5], &seeds))
            Py_RETURN_NONE;
        const at::Tensor* x = plain_tensor(a[3], width_of(prm.ell));
        if (!x) Py_RETURN_NONE;
        const int64_t n = x->numel(), shape[2] = {words_of(prm), n};
        void *stream, *msg;
        Result r;
        if (!take_stream(a[8], *x, &stream) || !take_output(a[7], *x, shape, at::kInt, 4, shape[0] * n, &r.o, &msg))
            Py_RETURN_NONE;
        const at::Tensor& m = THPVariable_Unpack(r.o);
        if (m.dim() != 2 || m.size(0) != shape[0] || m.size(1) != n) Py_RETURN_NONE;
        const void* p = x->data_ptr();
        return conclude(r, unlocked([&] {
            return reinterpret_cast<SendFn>(fn)(party, p, static_cast<uint32_t*>(msg), (uint64_t)n, &prm, &seeds, base, stream);
        }), a[1]);
    });
}

// reply(fn, name, msg0, msg1, params, seeds, elem_base, out, stream)
PyObject* py_reply(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn, base;
        bc_drelu_params prm;
        bc_seeds seeds;
        if (nargs != 9 || !as_u64(a[0], &fn) || !as_u64(a[6], &base) || !take_struct(a[4], &prm) || !take_struct(a[5], &seeds) ||
            (a[7] != Py_None && (!PyTuple_CheckExact(a[7]) || PyTuple_GET_SIZE(a[7]) != 2)))
            Py_RETURN_NONE;
        const at::Tensor *m0 = plain_tensor(a[2], 4), *m1 = plain_tensor(a[3], 4);
        if (!m0 || !m1 || m0->dim() != 2 || m0->sizes() != m1->sizes() || m0->size(0) != words_of(prm)) Py_RETURN_NONE;
        const int64_t n = m0->size(1);
        const uint32_t w = width_of(prm.ell);
        void *stream, *d0, *d1;
        Result r0, r1, r;
        const bool fresh = a[7] == Py_None;
        if (!take_stream(a[8], *m0, &stream) ||
            !take_output(fresh ? Py_None : PyTuple_GET_ITEM(a[7], 0), *m0, {n}, ring_type(w), w, n, &r0.o, &d0) ||
            !take_output(fresh ? Py_None : PyTuple_GET_ITEM(a[7], 1), *m0, {n}, ring_type(w), w, n, &r1.o, &d1))
            Py_RETURN_NONE;
        r.o = PyTuple_Pack(2, r0.o, r1.o);
        if (!r.o) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
        const auto *p0 = static_cast<const uint32_t*>(m0->data_ptr()), *p1 = static_cast<const uint32_t*>(m1->data_ptr());
        return conclude(r, unlocked([&] {
            return reinterpret_cast<ReplyFn>(fn)(p0, p1, d0, d1, (uint64_t)n, &prm, &seeds, base, stream);
        }), a[1]);
    });
}

// finish(fn, name, party, d, params, seeds, elem_base, out, stream)
PyObject* py_finish(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
    return guarded([&]() -> PyObject* {
        uint64_t fn, base;
        uint32_t party;
        bc_drelu_params prm;
        bc_seeds seeds;
        if (nargs != 9 || !as_u64(a[0], &fn) || !as_u32(a[2], &party) || !as_u64(a[6], &base) || !take_struct(a[4], &prm) ||
            !take_struct(a[5], &seeds))
            Py_RETURN_NONE;
        const uint32_t w = width_of(prm.ell);
        const at::Tensor* d = plain_tensor(a[3], w);
        if (!d) Py_RETURN_NONE;
        void *stream, *y;
        Result r;
        if (!take_stream(a[8], *d, &stream) || !take_output(a[7], *d, d->sizes(), ring_type(w), w, d->numel(), &r.o, &y))
            Py_RETURN_NONE;
        const void* p = d->data_ptr();
        const uint64_t n = (uint64_t)d->numel();
        return conclude(r, unlocked([&] {
            return reinterpret_cast<FinishFn>(fn)(party, p, y, n, &prm, &seeds, base, stream);
        }), a[1]);
    });
}

// set_check(f): f(rc, where) raises the binding's exception
PyObject* py_set_check(PyObject*, PyObject* f) {
    Py_INCREF(f);
    Py_XDECREF(g_check);
    g_check = f;
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"drelu", (PyCFunction)(void (*)(void))py_drelu, METH_FASTCALL, nullptr},
    {"trunc", (PyCFunction)(void (*)(void))py_trunc, METH_FASTCALL, nullptr},
    {"cut", (PyCFunction)(void (*)(void))py_cut, METH_FASTCALL, nullptr},
    {"rss", (PyCFunction)(void (*)(void))py_rss, METH_FASTCALL, nullptr},
    {"mul", (PyCFunction)(void (*)(void))py_mul, METH_FASTCALL, nullptr},
    {"send", (PyCFunction)(void (*)(void))py_send, METH_FASTCALL, nullptr},
    {"reply", (PyCFunction)(void (*)(void))py_reply, METH_FASTCALL, nullptr},
    {"finish", (PyCFunction)(void (*)(void))py_finish, METH_FASTCALL, nullptr},
    {"set_check", py_set_check, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
    g_struct = PyUnicode_InternFromString("_c");
    g_c = PyUnicode_InternFromString("c");
    g_stream = PyUnicode_InternFromString("cuda_stream");
    if (!g_struct || !g_c || !g_stream) return nullptr;
    return PyModule_Create(&kModule);
}
