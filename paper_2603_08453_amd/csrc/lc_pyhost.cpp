// CPython module _lychee_host: the host-side loops of the binding that Python would run element by element.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "lc_chunker.h"

namespace {

// UTF-8 bytes of a plain str where the object holds them (an ASCII str is its own UTF-8; others cache theirs).
inline bool str_text(PyObject* t, LcTokenText* out) {
    if (PyUnicode_IS_COMPACT_ASCII(t)) {
        *out = {reinterpret_cast<const char*>(PyUnicode_1BYTE_DATA(t)), PyUnicode_GET_LENGTH(t)};
        return true;
    }
    Py_ssize_t len = 0;
    const char* const p = PyUnicode_AsUTF8AndSize(t, &len);
    *out = {p, len};
    return p != nullptr;
}

// Levels of the tokens of one call, by object: where the tokens are looked up in a vocabulary the same str object comes
// again and again, and a separator test costs a few mispredicted branches (26 ns against 3 ns for the look-up).
// Direct-mapped; a miss computes the level, and a tokenizer that makes a str per token misses nearly always.
// 32768 tokens: 53 us as 37 objects, 109 us as 32768 objects of the same texts, 249 us from a vocabulary of 50000
// (its texts are not in the processor's caches either); 2.95 ms with an encode() and an offset per token in Python.
class LevelMemo {
  public:
    LevelMemo() : slot_() {}
    template <typename TextF>
    int level(const void* key, TextF text) {
        const uintptr_t u = reinterpret_cast<uintptr_t>(key) >> 4;
        Slot& s = slot_[(u ^ (u >> 10)) & (N - 1)];
        if (s.key != key) { s.key = key; s.level = lc_separator_level(text()); }
        return s.level;
    }

  private:
    static constexpr int N = 1024;
    struct Slot { const void* key; int level; };
    Slot slot_[N];
};

// chunk_tokens(tokens, min_len, max_len) -> list of boundaries, or a negative LC_ERR_* code.
// The tokens' bytes are read where the objects hold them: no concatenated copy, no offset array, and
// apart from a check of every object only the tokens inside the search windows are looked at.  The interpreter stays
// locked throughout (the bytes belong to the caller's objects).
PyObject* chunk_tokens(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
    if (n_args != 3) {
        PyErr_SetString(PyExc_TypeError, "chunk_tokens(tokens, min_len, max_len)");
        return nullptr;
    }
    const long min_len = PyLong_AsLong(args[1]), max_len = PyLong_AsLong(args[2]);
    if (PyErr_Occurred()) return nullptr;
    // (before the items are looked at: a new list can run the cyclic collector, and that any Python code, also such as
    // changes the caller's list; nothing between here and the cuts does)
    PyObject* out = PyList_New(0);
    PyObject* seq = out ? PySequence_Fast(args[0], "tokens must be a sequence") : nullptr;
    if (!seq) {
        Py_XDECREF(out);
        return nullptr;
    }
    Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
    PyObject** items = PySequence_Fast_ITEMS(seq);
    bool plain = true;                               // every token is a plain str, which no Python code can touch here
    LcTokenText unused;
    for (Py_ssize_t i = 0; i < n && plain; ++i) {
        plain = PyUnicode_CheckExact(items[i]);
        if (plain && !PyUnicode_IS_COMPACT_ASCII(items[i]) && !str_text(items[i], &unused)) {
            Py_DECREF(seq);
            Py_DECREF(out);
            return nullptr;
        }
    }
    if (!plain) {                                    // other objects: a tuple of what their encode() gives
        Py_SETREF(seq, PySequence_Tuple(seq));
        if (!seq) {
            Py_DECREF(out);
            return nullptr;
        }
        n = PyTuple_GET_SIZE(seq);
        PyObject* enc = PyTuple_New(n);
        for (Py_ssize_t i = 0; enc && i < n; ++i) {
            PyObject* const b = PyObject_CallMethod(PyTuple_GET_ITEM(seq, i), "encode", "s", "utf-8");
            if (b && !PyBytes_Check(b)) {
                PyErr_SetString(PyExc_TypeError, "encode() did not return bytes");
                Py_DECREF(b);
                Py_CLEAR(enc);
            } else if (!b) {
                Py_CLEAR(enc);
            } else {
                PyTuple_SET_ITEM(enc, i, b);
            }
        }
        Py_SETREF(seq, enc);
        if (!seq) {
            Py_DECREF(out);
            return nullptr;
        }
        items = PySequence_Fast_ITEMS(seq);
    }
    if (n > 0x7fffffff || min_len < 1 || max_len < min_len) {
        Py_SETREF(out, PyLong_FromLong(LC_ERR_INVALID_ARG));
    } else {
        LevelMemo memo;
        PyObject* const zero = PyLong_FromLong(0);
        bool ok = zero && PyList_Append(out, zero) == 0;
        Py_XDECREF(zero);
        ok = ok && lc_chunk_cuts(
            n, min_len, max_len,
            [&](int64_t i) {
                PyObject* const t = items[i];
                return memo.level(t, [&] {
                    LcTokenText x;
                    if (plain) (void)str_text(t, &x);          // (has worked before)
                    else x = {PyBytes_AS_STRING(t), PyBytes_GET_SIZE(t)};
                    return x;
                });
            },
            [&](int64_t end) {
                PyObject* const v = PyLong_FromLongLong(end);
                const bool in = v && PyList_Append(out, v) == 0;
                Py_XDECREF(v);
                return in;
            });
        if (!ok) Py_CLEAR(out);
    }
    Py_DECREF(seq);
    return out;
}

PyMethodDef methods[] = {
    {"chunk_tokens", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(chunk_tokens)), METH_FASTCALL,
     "chunk_tokens(tokens, min_len, max_len) -> boundaries, or a negative error code"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lychee_host", "Host-side loops of the binding.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lychee_host() { return PyModule_Create(&module); }
