// The per-layer calls of a decode loop as a CPython extension: argument marshalling of binding.py in C, for the argument
// types such a loop passes (tensors, addresses, None, plain numbers).  A ctypes call with fifteen converted arguments and the
// Python around it cost 5 us of host time in front of a launch of 2.5 us, more than a small launch takes on the device (four
// contexts of 17..128 rows, 16 x 256: 6.0 us); this way it is 0.6.  The prompt rows of four newcomers
// (s3_kv_fill_batch): 9.5 us a layer of host time, now 4.6.  Whatever else is passed comes back as None, and
// binding.py takes its ctypes path, which defines what is accepted.  Host code only; the library is called by address.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*step_fn)(void *, int32_t, int32_t, const int32_t *, const int32_t *, const void *, const void *, const void *, const void *,
                       const void *, void *, int32_t, float, void *, void *);
typedef int (*append_fn)(void *, int32_t, int32_t, const int32_t *, const int32_t *, const void *, const void *, const void *, const void *,
                         void *);
typedef int (*attention_fn)(void *, int32_t, int32_t, const void *, const void *, const void *, void *, int32_t, float, void *);

typedef int (*fill_fn)(void *, int32_t, int32_t, const int32_t *, const int32_t *, void **, void **, int32_t, void *, void *, const int32_t *,
                       void *);

static step_fn g_step, g_static;
static fill_fn g_fill;
static append_fn g_append;
static attention_fn g_attention;
static PyObject *s_data_ptr, *s_value;
static PyObject *g_void_p;  // the type ctypes.c_void_p

// 1: converted; 0: a type that is left to the ctypes path; -1: a Python error is set.
static int address(PyObject *x, void **out) {
    if (x == Py_None) {
        *out = nullptr;
        return 1;
    }
    PyObject *owned = nullptr;
    if (!PyLong_Check(x)) {
        owned = PyObject_CallMethodNoArgs(x, s_data_ptr);
        if (!owned) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
            PyErr_Clear();
            return 0;
        }
        x = owned;
    }
    const bool ok = PyLong_Check(x);
    if (ok) *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(x);
    Py_XDECREF(owned);
    return PyErr_Occurred() ? -1 : ok;
}

// An arena: a ctypes.c_void_p and nothing else that has a `value` (other ctypes numbers, enum members: the ctypes path refuses them).
static int handle(PyObject *x, void **out) {
    if ((PyObject *)Py_TYPE(x) != g_void_p) return 0;
    PyObject *v = PyObject_GetAttr(x, s_value);
    if (!v) return -1;
    const bool ok = PyLong_Check(v);  // (a null pointer's is None)
    if (ok) *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    return PyErr_Occurred() ? -1 : ok;
}

static int number(PyObject *x, int32_t *out) {
    if (!PyLong_Check(x)) return 0;
    *out = (int32_t)PyLong_AsUnsignedLongMask(x);
    return PyErr_Occurred() ? -1 : 1;
}

static int real(PyObject *x, float *out) {
    if (!PyFloat_CheckExact(x)) return 0;
    *out = (float)PyFloat_AS_DOUBLE(x);
    return 1;
}

static int stream_of(PyObject *x, void **out) { return x == Py_None || PyLong_Check(x) ? address(x, out) : 0; }

#define TAKE(expr)                            \
    do {                                      \
        const int rc_ = (expr);               \
        if (rc_ < 0) return nullptr;          \
        if (rc_ == 0) Py_RETURN_NONE;         \
    } while (0)

// (arena, layer, n, slot_off, pos, q, k_new, v_new, out, out_dtype, scale, len_out, stream)
static PyObject *call_step(step_fn fn, PyObject *const *a, Py_ssize_t count) {
    if (!fn || count != 13) Py_RETURN_NONE;
    void *arena, *p[6], *len_out, *stream;
    int32_t layer, n, dtype;
    float scale;
    TAKE(handle(a[0], &arena));
    TAKE(number(a[1], &layer));
    TAKE(number(a[2], &n));
    for (int i = 0; i < 6; i++) TAKE(address(a[3 + i], &p[i]));
    TAKE(number(a[9], &dtype));
    TAKE(real(a[10], &scale));
    TAKE(address(a[11], &len_out));
    TAKE(stream_of(a[12], &stream));
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = fn(arena, layer, n, nullptr, nullptr, p[0], p[1], p[2], p[3], p[4], p[5], dtype, scale, len_out, stream);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
}
static PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t count) { return call_step(g_step, a, count); }
static PyObject *step_static(PyObject *, PyObject *const *a, Py_ssize_t count) { return call_step(g_static, a, count); }

// (arena, layer, n, slot_off, pos, k_new, v_new, stream)
static PyObject *append(PyObject *, PyObject *const *a, Py_ssize_t count) {
    if (!g_append || count != 8) Py_RETURN_NONE;
    void *arena, *p[4], *stream;
    int32_t layer, n;
    TAKE(handle(a[0], &arena));
    TAKE(number(a[1], &layer));
    TAKE(number(a[2], &n));
    for (int i = 0; i < 4; i++) TAKE(address(a[3 + i], &p[i]));
    TAKE(stream_of(a[7], &stream));
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = g_append(arena, layer, n, nullptr, nullptr, p[0], p[1], p[2], p[3], stream);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
}

// (arena, layer, n, q, slot_off, cur_len, out, out_dtype, scale, stream)
static PyObject *attention(PyObject *, PyObject *const *a, Py_ssize_t count) {
    if (!g_attention || count != 10) Py_RETURN_NONE;
    void *arena, *p[4], *stream;
    int32_t layer, n, dtype;
    float scale;
    TAKE(handle(a[0], &arena));
    TAKE(number(a[1], &layer));
    TAKE(number(a[2], &n));
    for (int i = 0; i < 4; i++) TAKE(address(a[3 + i], &p[i]));
    TAKE(number(a[7], &dtype));
    TAKE(real(a[8], &scale));
    TAKE(stream_of(a[9], &stream));
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = g_attention(arena, layer, n, p[0], p[1], p[2], p[3], dtype, scale, stream);
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(rc);
}

// Contiguous 32-bit whole numbers, and how many; 0: something else.
static int numbers(PyObject *x, Py_buffer *view, Py_ssize_t *count) {
    if (!PyObject_CheckBuffer(x)) return 0;
    if (PyObject_GetBuffer(x, view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
        PyErr_Clear();
        return 0;
    }
    if (view->ndim == 1 && view->itemsize == 4 && view->format && view->format[0] == 'i' && !view->format[1]) {
        *count = view->shape[0];
        return 1;
    }
    PyBuffer_Release(view);
    return 0;
}

// (arena, layer, slot_ids, n_rows, k_rows, v_rows, stream)
static PyObject *fill(PyObject *, PyObject *const *a, Py_ssize_t count) {
    constexpr Py_ssize_t MOST = 256;
    if (!g_fill || count != 7 || !PyList_Check(a[4]) || !PyList_Check(a[5])) Py_RETURN_NONE;
    const Py_ssize_t n = PyList_GET_SIZE(a[4]);
    if (n > MOST || PyList_GET_SIZE(a[5]) != n) Py_RETURN_NONE;
    void *arena, *stream, *rows[2][MOST];
    int32_t layer;
    TAKE(handle(a[0], &arena));
    TAKE(number(a[1], &layer));
    TAKE(stream_of(a[6], &stream));
    for (int w = 0; w < 2; w++)
        for (Py_ssize_t i = 0; i < n; i++) {
            if (i >= PyList_GET_SIZE(a[4 + w])) Py_RETURN_NONE;  // (a data_ptr() that shortened the list)
            TAKE(address(PyList_GET_ITEM(a[4 + w], i), &rows[w][i]));
        }
    Py_buffer ids, lens;
    Py_ssize_t n_ids = -1, n_lens = -1;
    TAKE(numbers(a[2], &ids, &n_ids));
    if (numbers(a[3], &lens, &n_lens) == 0) {
        PyBuffer_Release(&ids);
        Py_RETURN_NONE;
    }
    int rc = 0;
    const bool fits = n_ids == n && n_lens >= n;
    if (fits) {
        Py_BEGIN_ALLOW_THREADS;
        rc = g_fill(arena, layer, (int32_t)n, (const int32_t *)ids.buf, (const int32_t *)lens.buf, rows[0], rows[1], 0, nullptr, nullptr,
                    nullptr, stream);
        Py_END_ALLOW_THREADS;
    }
    PyBuffer_Release(&ids);
    PyBuffer_Release(&lens);
    if (!fits) Py_RETURN_NONE;
    return PyLong_FromLong(rc);
}

// (ctypes.c_void_p, then the addresses of s3_decode_step, s3_decode_step_static, s3_kv_append, s3_decode_attention and
// s3_kv_fill_batch of the loaded library)
static PyObject *connect(PyObject *, PyObject *args) {
    unsigned long long s, t, p, q, f;
    PyObject *type;
    if (!PyArg_ParseTuple(args, "O!KKKKK", &PyType_Type, &type, &s, &t, &p, &q, &f)) return nullptr;
    Py_INCREF(type);
    Py_XSETREF(g_void_p, type);
    g_step = (step_fn)(uintptr_t)s;
    g_static = (step_fn)(uintptr_t)t;
    g_append = (append_fn)(uintptr_t)p;
    g_attention = (attention_fn)(uintptr_t)q;
    g_fill = (fill_fn)(uintptr_t)f;
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"connect", connect, METH_VARARGS, nullptr},
    {"step", (PyCFunction)(void (*)())step, METH_FASTCALL, nullptr},
    {"step_static", (PyCFunction)(void (*)())step_static, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void (*)())append, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void (*)())attention, METH_FASTCALL, nullptr},
    {"fill", (PyCFunction)(void (*)())fill, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "_s3call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

PyMODINIT_FUNC PyInit__s3call() {
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_value = PyUnicode_InternFromString("value");
    if (!s_data_ptr || !s_value) return nullptr;
    return PyModule_Create(&module);
}
