// CPython module _lychee_torch: argument marshalling of the per-token entry points for torch tensors.
//
// A decode step at a short context is shorter on the GPU than its call was in Python: ctypes
// conversions, tensor accessors and the current-stream object took about half of the 12.9 us a call spent on the
// host.  Here the tensors are read through torch's C++ objects.  The module calls the C ABI through the
// addresses the binding hands over (bind), so it works with whichever build of the library is loaded.
// A call with arguments that are no tensors returns NotImplemented and the binding marshals it itself.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <exception>

#include "lychee.h"

namespace {

decltype(&lc_decode_step) g_decode_step = nullptr;
decltype(&lc_decode_step_static) g_decode_step_static = nullptr;
decltype(&lc_retrieve) g_retrieve = nullptr;
decltype(&lc_sparse_decode) g_sparse_decode = nullptr;
decltype(&lc_append) g_append = nullptr;

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) {
        PyErr_SetString(PyExc_TypeError, "bind(decode_step, decode_step_static, retrieve, sparse_decode, append)");
        return nullptr;
    }
    g_decode_step = reinterpret_cast<decltype(g_decode_step)>(PyLong_AsVoidPtr(a[0]));
    g_decode_step_static = reinterpret_cast<decltype(g_decode_step_static)>(PyLong_AsVoidPtr(a[1]));
    g_retrieve = reinterpret_cast<decltype(g_retrieve)>(PyLong_AsVoidPtr(a[2]));
    g_sparse_decode = reinterpret_cast<decltype(g_sparse_decode)>(PyLong_AsVoidPtr(a[3]));
    g_append = reinterpret_cast<decltype(g_append)>(PyLong_AsVoidPtr(a[4]));
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

// Positional arguments of one call.
class Args {
  public:
    Args(PyObject* const* a, Py_ssize_t n) : a_(a), n_(n) {}
    bool count(Py_ssize_t n) {
        if (n_ == n) return true;
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", n, n_);
        return false;
    }
    // The tensor at i, or null for None; anything else makes the call not ours.
    const at::Tensor* tensor(int i) {
        if (a_[i] == Py_None) return nullptr;
        if (!THPVariable_Check(a_[i])) { foreign_ = true; return nullptr; }
        return &THPVariable_Unpack(a_[i]);
    }
    void* ptr(int i) {
        const at::Tensor* t = tensor(i);
        return t ? t->data_ptr() : nullptr;
    }
    // What int(x) gives, in C's int (as ctypes passes it: the low 32 bits).
    int integer(int i) {
        PyObject* const v = PyLong_CheckExact(a_[i]) ? Py_NewRef(a_[i]) : PyNumber_Long(a_[i]);
        const int r = v ? (int)PyLong_AsUnsignedLongMask(v) : -1;
        Py_XDECREF(v);
        return r;
    }
    // The same of an integer alone; a float or a text makes the call not ours (ctypes refuses it).
    int whole(int i) {
        if (!PyIndex_Check(a_[i])) { foreign_ = true; return -1; }
        PyObject* const v = PyNumber_Index(a_[i]);
        const int r = v ? (int)PyLong_AsUnsignedLongMask(v) : -1;
        Py_XDECREF(v);
        return r;
    }
    lc_index* handle(int i) { return static_cast<lc_index*>(PyLong_AsVoidPtr(a_[i])); }
    void* stream(int i) {
        if (a_[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject* const v = PyObject_GetAttrString(a_[i], "cuda_stream");
        void* const s = v ? PyLong_AsVoidPtr(v) : nullptr;
        Py_XDECREF(v);
        return s;
    }
    PyObject* operator[](int i) const { return a_[i]; }
    bool foreign() const { return foreign_; }

  private:
    PyObject* const* a_;
    Py_ssize_t n_;
    bool foreign_ = false;
};

bool cache_strides(const at::Tensor& K, const at::Tensor& V, bool shapes, int64_t (&s)[3]) {
    if ((shapes && !K.sizes().equals(V.sizes())) || !K.strides().equals(V.strides())) {
        PyErr_SetString(PyExc_AssertionError, "K and V must have the same shape and strides");
        return false;
    }
    if (K.dim() != 4 || K.stride(3) != 1) {
        PyErr_SetString(PyExc_AssertionError, "cache must be [B][H_kv][tokens][d] with d contiguous");
        return false;
    }
    for (int i = 0; i < 3; ++i) s[i] = K.stride(i);
    return true;
}
// The interpreter is free for other threads while a call is in the library, as it is under ctypes: a launch can block
// (a full hardware queue).  Everything the call needs has been read from the Python objects before.
class Unlocked {
  public:
    Unlocked() : state_(PyEval_SaveThread()) {}
    ~Unlocked() { PyEval_RestoreThread(state_); }
    Unlocked(const Unlocked&) = delete;
    Unlocked& operator=(const Unlocked&) = delete;

  private:
    PyThreadState* state_;
};
size_t bytes(const at::Tensor& t) { return (size_t)t.numel() * t.element_size(); }

// The result of a call, or NotImplemented / the pending Python error.
template <typename F>
PyObject* guarded(Args& a, F call) {
    try {
        int rc = 0;
        const bool done = call(&rc);
        if (PyErr_Occurred()) return nullptr;
        if (a.foreign() || !done) Py_RETURN_NOTIMPLEMENTED;
        return PyLong_FromLong(rc);
    } catch (const std::exception& e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// decode_step(handle, q, K, V, budget, out, ws or None, lse, chunk_ids, counts, stream, static)
PyObject* decode_step(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a(args, n);
    if (!a.count(12)) return nullptr;
    return guarded(a, [&](int* rc) {
        const at::Tensor *q = a.tensor(1), *K = a.tensor(2), *V = a.tensor(3), *ws = a.tensor(6), *ids = a.tensor(8);
        const bool fixed = a[11] == Py_True;
        if (!q || !K || !V || (!fixed && !ws) || a.foreign()) return false;
        int64_t s[3];
        if (!cache_strides(*K, *V, true, s)) return true;
        const int budget = a.integer(4), cap = ids ? (int)ids->size(-1) : 0;
        float* const out = static_cast<float*>(a.ptr(5));
        float* const lse = static_cast<float*>(a.ptr(7));
        int32_t* const counts = static_cast<int32_t*>(a.ptr(9));
        if (PyErr_Occurred() || a.foreign()) return false;
        int32_t* const idp = ids ? static_cast<int32_t*>(ids->data_ptr()) : nullptr;
        void* const st = a.stream(10);
        if (PyErr_Occurred()) return false;
        lc_index* const idx = a.handle(0);
        if (PyErr_Occurred()) return false;
        const void *qd = q->data_ptr(), *kd = K->data_ptr(), *vd = V->data_ptr();
        void* const wd = fixed ? nullptr : ws->data_ptr();
        const size_t wn = fixed ? 0 : bytes(*ws);
        const int H_q = (int)q->size(1);
        const Unlocked unlocked;
        *rc = fixed ? g_decode_step_static(idx, qd, kd, vd, s, H_q, budget, out, lse, idp, counts, cap, st)
                    : g_decode_step(idx, qd, kd, vd, s, H_q, budget, out, lse, idp, counts, cap, wd, wn, st);
        return true;
    });
}

// retrieve(handle, q, budget, chunk_ids, counts, ws, scores, stream)
PyObject* retrieve(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a(args, n);
    if (!a.count(8)) return nullptr;
    return guarded(a, [&](int* rc) {
        const at::Tensor *q = a.tensor(1), *ids = a.tensor(3), *ws = a.tensor(5);
        if (!q || !ids || !ws || a.foreign()) return false;
        const int budget = a.whole(2);
        int32_t* const counts = static_cast<int32_t*>(a.ptr(4));
        float* const scores = static_cast<float*>(a.ptr(6));
        if (PyErr_Occurred() || a.foreign()) return false;
        void* const st = a.stream(7);
        if (PyErr_Occurred()) return false;
        lc_index* const idx = a.handle(0);
        if (PyErr_Occurred()) return false;
        const void* const qd = q->data_ptr();
        int32_t* const idp = static_cast<int32_t*>(ids->data_ptr());
        const int H_q = (int)q->size(1), cap = (int)ids->size(2);
        void* const wd = ws->data_ptr();
        const size_t wn = bytes(*ws);
        const Unlocked unlocked;
        *rc = g_retrieve(idx, qd, H_q, budget, idp, counts, scores, cap, wd, wn, st);
        return true;
    });
}

// sparse_decode(handle, q, K, V, chunk_ids, counts, out, ws, lse, stream)
PyObject* sparse_decode(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a(args, n);
    if (!a.count(10)) return nullptr;
    return guarded(a, [&](int* rc) {
        const at::Tensor *q = a.tensor(1), *K = a.tensor(2), *V = a.tensor(3), *ids = a.tensor(4), *ws = a.tensor(7);
        if (!q || !K || !V || !ids || !ws || a.foreign()) return false;
        int64_t s[3];
        if (!cache_strides(*K, *V, false, s)) return true;
        const int32_t* const counts = static_cast<const int32_t*>(a.ptr(5));
        float* const out = static_cast<float*>(a.ptr(6));
        float* const lse = static_cast<float*>(a.ptr(8));
        if (a.foreign()) return false;
        void* const st = a.stream(9);
        if (PyErr_Occurred()) return false;
        lc_index* const idx = a.handle(0);
        if (PyErr_Occurred()) return false;
        const void *qd = q->data_ptr(), *kd = K->data_ptr(), *vd = V->data_ptr();
        const int32_t* const idp = static_cast<const int32_t*>(ids->data_ptr());
        const int H_q = (int)q->size(1), cap = (int)ids->size(2);
        void* const wd = ws->data_ptr();
        const size_t wn = bytes(*ws);
        const Unlocked unlocked;
        *rc = g_sparse_decode(idx, qd, kd, vd, s, idp, counts, cap, H_q, out, lse, wd, wn, st);
        return true;
    });
}

// append(handle, K, V, k_new, v_new, close flags or None, ws, stream)
PyObject* append(PyObject*, PyObject* const* args, Py_ssize_t n) {
    Args a(args, n);
    if (!a.count(8)) return nullptr;
    return guarded(a, [&](int* rc) {
        const at::Tensor *K = a.tensor(1), *V = a.tensor(2), *k = a.tensor(3), *v = a.tensor(4), *ws = a.tensor(6);
        if (!K || !V || !k || !v || !ws || a.foreign()) return false;
        int64_t s[3];
        if (!cache_strides(*K, *V, false, s)) return true;
        uint8_t flags[1024] = {};                            // lc_append takes at most 1024 sequences
        const bool given = a[5] != Py_None;
        if (given) {
            // (a tuple of its own: telling whether an element is true can run code that changes the caller's list)
            PyObject* const seq = PyObject_Size(a[5]) >= 0 ? PySequence_Tuple(a[5]) : nullptr;
            if (!seq) return false;
            const Py_ssize_t m = PyTuple_GET_SIZE(seq);
            bool ok = m <= (Py_ssize_t)sizeof(flags);
            for (Py_ssize_t i = 0; ok && i < m; ++i) {
                const int t = PyObject_IsTrue(PyTuple_GET_ITEM(seq, i));
                if (t < 0) ok = false;
                else flags[i] = (uint8_t)t;
            }
            Py_DECREF(seq);
            if (!ok) return false;
        }
        void* const st = a.stream(7);
        if (PyErr_Occurred()) return false;
        lc_index* const idx = a.handle(0);
        if (PyErr_Occurred()) return false;
        void *kd = K->data_ptr(), *vd = V->data_ptr();
        const void *kn = k->data_ptr(), *vn = v->data_ptr();
        void* const wd = ws->data_ptr();
        const size_t wn = bytes(*ws);
        const Unlocked unlocked;
        *rc = g_append(idx, kd, vd, s, kn, vn, given ? flags : nullptr, wd, wn, st);
        return true;
    });
}

template <typename F>
PyCFunction fast(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef methods[] = {
    {"bind", fast(bind), METH_FASTCALL, "addresses of the library's entry points"},
    {"decode_step", fast(decode_step), METH_FASTCALL, ""},
    {"retrieve", fast(retrieve), METH_FASTCALL, ""},
    {"sparse_decode", fast(sparse_decode), METH_FASTCALL, ""},
    {"append", fast(append), METH_FASTCALL, ""},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lychee_torch", "Tensor marshalling of the per-token entry points.", -1,
                      methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lychee_torch() { return PyModule_Create(&module); }
