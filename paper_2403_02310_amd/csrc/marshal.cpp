// Python module _marshal: the argument marshalling of the two attention calls that a scheduling iteration makes for every layer.
// Through ctypes it kept the host busy for 8 to 11 us a call, most of the 24 to 27 us that a small batch took from pass to pass
// (64 tokens next to three decodes, 4 heads and one; 12.2 us so); here it takes 2.  Conversions that need more than a look at the object (a list of lengths, an array
// of another type, a wrong table) go through the functions that binding.py registers, which also raise its errors.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>
#include <vector>

namespace {

using AppendFn = int (*)(void *, const void *, const void *, void *, void *, const int32_t *, const int32_t *, const int32_t *, const int32_t *,
                         int32_t, int32_t, int64_t, void *, void *);
using AttentionFn = int (*)(void *, const void *, const void *, const void *, const int32_t *, const int32_t *, const int32_t *, const int32_t *,
                            int32_t, int32_t, int64_t, float, void *, void *, void *);
using NoallocFn = int (*)(void *, const void *, const void *, const void *, const int32_t *, const int32_t *, const int32_t *, const int32_t *,
                          int32_t, int32_t, int64_t, float, void *, void *);
AppendFn append_fn;
AttentionFn attention_fn;
NoallocFn noalloc_fn;
// registered by binding.py, kept for the life of the process
PyObject *ndarray_type, *as_i32, *current_stream, *refuse_table;
PyObject *as_c_int32, *as_c_int64, *as_c_address;
PyObject *s_is_contiguous, *s_data_ptr, *s_shape, *s_cuda_stream;

// An int as the C call takes it (wrapped to 64 bits), None and what is no int through `convert`, which takes and refuses what a
// ctypes call does; sets an error otherwise.
bool as_int(PyObject *o, PyObject *convert, uint64_t *out) {
    PyObject *made = nullptr;
    if (!PyLong_Check(o)) {
        if (!(made = PyObject_CallOneArg(convert, o))) return false;
        o = made;
    }
    const bool none = o == Py_None;  // a null address
    *out = none ? 0 : PyLong_AsUnsignedLongLongMask(o);
    Py_XDECREF(made);
    return none || !(*out == (uint64_t)-1 && PyErr_Occurred());
}
bool as_address(PyObject *o, void **out) {
    uint64_t v = 0;
    if (o != Py_None && !as_int(o, as_c_address, &v)) return false;
    *out = reinterpret_cast<void *>(v);
    return true;
}

// Address of a device tensor (contiguous), of an int, or null for None.
bool device(PyObject *t, void **out) {
    *out = nullptr;
    if (t == Py_None || PyLong_Check(t)) return as_address(t, out);
    PyObject *c = PyObject_CallMethodNoArgs(t, s_is_contiguous);
    if (!c) return false;
    const int yes = PyObject_IsTrue(c);
    Py_DECREF(c);
    if (yes < 0) return false;
    if (!yes) {
        PyErr_SetString(PyExc_ValueError, "device tensors must be contiguous");
        return false;
    }
    PyObject *address = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!address) return false;
    const bool ok = as_address(address, out);
    Py_DECREF(address);
    return ok;
}

// "i", or "=i" and "<i" as unaligned arrays and ctypes arrays have it (the host's bytes are little-endian).
static_assert(__BYTE_ORDER__ == __ORDER_LITTLE_ENDIAN__, "'<' names the host's byte order");
bool is_int32(const Py_buffer &view) {
    if (view.itemsize != 4 || !view.format) return false;
    const char *f = view.format;
    if (*f == '@' || *f == '=' || *f == '<') ++f;
    return (*f == 'i' || *f == 'l') && f[1] == 0;
}

// int32 lengths, contiguous: an array of that kind as it is, anything else through as_i32.
struct Lengths {
    Py_buffer view{};
    bool held = false;
    std::vector<int32_t> aligned;  // the lengths, if the buffer holds them at an odd address
    ~Lengths() {
        if (held) PyBuffer_Release(&view);
    }
    bool take(PyObject *a) {
        held = PyObject_GetBuffer(a, &view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) == 0;
        if (!held) return false;
        if (view.ndim >= 1 && is_int32(view)) {
            if (reinterpret_cast<uintptr_t>(view.buf) % alignof(int32_t) != 0) {
                aligned.resize(static_cast<size_t>(view.len) / sizeof(int32_t));
                std::memcpy(aligned.data(), view.buf, aligned.size() * sizeof(int32_t));
            }
            return true;
        }
        PyBuffer_Release(&view);
        held = false;
        return false;
    }
    bool get(PyObject *a) {
        if (PyObject_TypeCheck(a, reinterpret_cast<PyTypeObject *>(ndarray_type))) {
            if (take(a)) return true;
            PyErr_Clear();
        }
        PyObject *made = PyObject_CallOneArg(as_i32, a);
        if (!made) return false;
        const bool ok = take(made);  // the view holds the array
        Py_DECREF(made);
        if (!ok && !PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "lengths must convert to int32");
        return ok;
    }
    const int32_t *data() const { return aligned.empty() ? static_cast<const int32_t *>(view.buf) : aligned.data(); }
    int32_t count() const { return static_cast<int32_t>(view.shape[0]); }
    Py_ssize_t all() const { return view.len / 4; }
    int64_t sum() const {
        int64_t s = 0;
        for (Py_ssize_t i = 0; i < all(); ++i) s += data()[i];
        return s;
    }
};

// The block table must be [>= num_seqs, max_blocks]: the C call is given a bare pointer and walks it with the handle's row width.
bool table_fits(PyObject *table, int64_t max_blocks, int32_t num_seqs) {
    if (table == Py_None || PyLong_Check(table)) return true;
    PyObject *shape = PyObject_GetAttr(table, s_shape);
    bool fits = false;
    if (shape && PyTuple_Check(shape) && PyTuple_GET_SIZE(shape) == 2) {
        const int64_t rows = PyLong_AsLongLong(PyTuple_GET_ITEM(shape, 0)), width = PyLong_AsLongLong(PyTuple_GET_ITEM(shape, 1));
        fits = width == max_blocks && rows >= num_seqs;  // contiguity: device()
    }
    Py_XDECREF(shape);
    PyErr_Clear();
    if (fits) return true;
    PyObject *r = PyObject_CallFunction(refuse_table, "OLi", table, (long long)max_blocks, (int)num_seqs);
    Py_XDECREF(r);
    return r != nullptr;  // an object without a shape
}

bool stream_of(PyObject *s, void **out) {
    PyObject *v;
    if (s == Py_None) v = PyObject_CallNoArgs(current_stream);
    else if (PyLong_Check(s)) Py_INCREF(s), v = s;
    else v = PyObject_GetAttr(s, s_cuda_stream);
    if (!v) return false;
    const bool ok = as_address(v, out);
    Py_DECREF(v);
    return ok;
}

// What the three calls share.
struct Batch {
    Lengths q_start, q_len, ctx_len;
    int32_t num_seqs = 0, num_tokens = 0;
    int64_t num_pages = 0;
    void *table = nullptr;
    bool get(int64_t max_blocks, PyObject *block_table, PyObject *qs, PyObject *ql, PyObject *cl, PyObject *pages, PyObject *tokens, PyObject *k_cache) {
        if (!q_start.get(qs) || !q_len.get(ql) || !ctx_len.get(cl)) return false;
        num_seqs = q_len.count();
        if (q_start.all() < num_seqs || q_len.all() < num_seqs || ctx_len.all() < num_seqs) {
            PyErr_Format(PyExc_ValueError, "q_start, q_len and ctx_len need one for each sequence of q_len (%d), got %zd, %zd and %zd", (int)num_seqs,
                         q_start.all(), q_len.all(), ctx_len.all());
            return false;
        }
        uint64_t v;
        if (tokens == Py_None) num_tokens = static_cast<int32_t>(q_len.sum());
        else if (as_int(tokens, as_c_int32, &v)) num_tokens = static_cast<int32_t>(v);
        else return false;
        if (pages == Py_None) {
            PyObject *shape = PyObject_GetAttr(k_cache, s_shape);
            PyObject *first = shape ? PySequence_GetItem(shape, 0) : nullptr;
            PyObject *whole = first ? PyNumber_Long(first) : nullptr;
            const bool ok = whole && as_int(whole, as_c_int64, &v);
            Py_XDECREF(whole);
            Py_XDECREF(first);
            Py_XDECREF(shape);
            if (!ok) return false;
        } else if (!as_int(pages, as_c_int64, &v)) return false;
        num_pages = static_cast<int64_t>(v);
        return table_fits(block_table, max_blocks, num_seqs) && device(block_table, &table);
    }
};

bool arity(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, n);
    return false;
}

// (handle, max_blocks, k_new, v_new, k_cache, v_cache, block_table, q_start, q_len, ctx_len, num_pages, num_tokens, workspace, stream)
PyObject *kv_append(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!arity(n, 14)) return nullptr;
    void *h, *k_new, *v_new, *k_cache, *v_cache, *ws, *stream;
    Batch b;
    if (!device(a[0], &h) || !b.get(PyLong_AsLongLong(a[1]), a[6], a[7], a[8], a[9], a[10], a[11], a[4]) || !device(a[2], &k_new) ||
        !device(a[3], &v_new) || !device(a[4], &k_cache) || !device(a[5], &v_cache) || !device(a[12], &ws) || !stream_of(a[13], &stream))
        return nullptr;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = append_fn(h, k_new, v_new, k_cache, v_cache, static_cast<const int32_t *>(b.table), b.q_start.data(), b.q_len.data(), b.ctx_len.data(), b.num_seqs,
                   b.num_tokens, b.num_pages, ws, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// (handle, max_blocks, q, k_cache, v_cache, block_table, q_start, q_len, ctx_len, num_pages, num_tokens, sm_scale, out, stream[, workspace]):
// without a workspace the allocation-free call
PyObject *attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 14 && !arity(n, 15)) return nullptr;
    void *h, *q, *k_cache, *v_cache, *out, *stream, *ws = nullptr;
    Batch b;
    if (!device(a[0], &h) || !b.get(PyLong_AsLongLong(a[1]), a[5], a[6], a[7], a[8], a[9], a[10], a[3]) || !device(a[2], &q) || !device(a[3], &k_cache) ||
        !device(a[4], &v_cache))
        return nullptr;
    const float scale = static_cast<float>(PyFloat_AsDouble(a[11]));
    if (PyErr_Occurred() || !device(a[12], &out) || !stream_of(a[13], &stream) || (n == 15 && !device(a[14], &ws))) return nullptr;
    const auto *table = static_cast<const int32_t *>(b.table);
    int st;
    Py_BEGIN_ALLOW_THREADS
    if (n == 15)
        st = attention_fn(h, q, k_cache, v_cache, table, b.q_start.data(), b.q_len.data(), b.ctx_len.data(), b.num_seqs, b.num_tokens, b.num_pages, scale, out, ws, stream);
    else
        st = noalloc_fn(h, q, k_cache, v_cache, table, b.q_start.data(), b.q_len.data(), b.ctx_len.data(), b.num_seqs, b.num_tokens, b.num_pages, scale, out, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

void keep(PyObject **const *places, PyObject *const *objects, int n) {
    for (int i = 0; i < n; ++i) {
        Py_INCREF(objects[i]);
        Py_XSETREF(*places[i], objects[i]);
    }
}

// (address of sarathi_kv_append, .._hybrid_attention, .._hybrid_attention_noalloc, numpy.ndarray, as_i32, current_stream, refuse_table)
PyObject *setup(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!arity(n, 7)) return nullptr;
    void *f[3];
    for (int i = 0; i < 3; ++i)
        if (!as_address(a[i], &f[i])) return nullptr;
    if (!PyType_Check(a[3])) {
        PyErr_SetString(PyExc_TypeError, "the array type expected");
        return nullptr;
    }
    append_fn = reinterpret_cast<AppendFn>(f[0]);
    attention_fn = reinterpret_cast<AttentionFn>(f[1]);
    noalloc_fn = reinterpret_cast<NoallocFn>(f[2]);
    PyObject **const places[] = {&ndarray_type, &as_i32, &current_stream, &refuse_table};
    keep(places, a + 3, 4);
    Py_RETURN_NONE;
}

// (as_c_int32, as_c_int64, as_c_address)
PyObject *conversions(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (!arity(n, 3)) return nullptr;
    PyObject **const places[] = {&as_c_int32, &as_c_int64, &as_c_address};
    keep(places, a, 3);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"kv_append", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(kv_append)), METH_FASTCALL, nullptr},
    {"attention", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(attention)), METH_FASTCALL, nullptr},
    {"conversions", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(conversions)), METH_FASTCALL, nullptr},
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(setup)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Argument marshalling of libsarathi's calls.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_shape = PyUnicode_InternFromString("shape");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_is_contiguous || !s_data_ptr || !s_shape || !s_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
