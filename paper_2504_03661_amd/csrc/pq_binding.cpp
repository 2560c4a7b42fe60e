// The per-step calls of the Python binding (pq_attn_decode, pq_encode_append) without ctypes: arguments are taken apart
// here, the library's functions are called through the addresses that binding.py hands over.  A decoding step of one
// short sequence (32 heads, 1K tokens) is bound by the host: with ctypes the two calls took 13 us of the step, marshalling
// ten pointers each through Python helpers; with this module the step takes 16.1 us, before 22.8.
//
// As binding.py's helpers do it: a pointer argument is None (NULL), an int, or an object with data_ptr(); a stream is
// None (torch's current stream, through the callable handed over), an int, or an object with a cuda_stream attribute.
// The calls run without the interpreter lock and return the library's status.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

namespace {

typedef int (*decode_fn)(void *, const void *, const uint8_t *, const uint8_t *, const int32_t *, const void *, const void *,
                         const void *, const void *, const int32_t *, float, float *, void *);
typedef int (*append_fn)(void *, const void *, const void *, int32_t, const void *, const void *, uint8_t *, uint8_t *,
                         int32_t *, void *);

PyObject *s_data_ptr, *s_cuda_stream, *s_value;

// false: a Python exception is set
bool pointer(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    if (PyLong_Check(o)) {
        *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
        return !PyErr_Occurred();
    }
    PyObject *p = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (p == nullptr)
        return false;
    PyObject *n = PyNumber_Long(p);
    Py_DECREF(p);
    if (n == nullptr)
        return false;
    *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return !PyErr_Occurred();
}

// the context: None, an int, or a ctypes.c_void_p (binding.py hands over no other)
bool handle(PyObject *o, void **out)
{
    if (o == Py_None || PyLong_Check(o))
        return pointer(o, out);
    PyObject *v = PyObject_GetAttr(o, s_value);
    if (v == nullptr)
        return false;
    const bool ok = pointer(v, out);
    Py_DECREF(v);
    return ok;
}

bool integer(PyObject *o, uint64_t *out)
{
    PyObject *n = PyNumber_Long(o);
    if (n == nullptr)
        return false;
    *out = PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return !PyErr_Occurred();
}

// `current`: called for None; returns the raw stream as an int
bool stream(PyObject *o, PyObject *current, void **out)
{
    PyObject *v = o == Py_None ? PyObject_CallNoArgs(current) : PyLong_Check(o) ? Py_NewRef(o) : PyObject_GetAttr(o, s_cuda_stream);
    if (v == nullptr)
        return false;
    uint64_t n = 0;
    const bool ok = integer(v, &n);
    Py_DECREF(v);
    *out = (void *)(uintptr_t)n;
    return ok;
}

bool count(Py_ssize_t n, Py_ssize_t want)
{
    if (n != want)
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return n == want;
}

// decode(function address, current-stream callable, <the 13 arguments of pq_attn_decode>)
PyObject *decode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *f, *p[11], *s;
    if (!count(n, 15) || !pointer(a[0], &f) || !handle(a[2], &p[0]))
        return nullptr;
    for (int i = 1; i < 10; ++i)  // q, k_codes, v_codes, ctx_len, k_codebook, v_codebook, recent_k, recent_v, recent_len
        if (!pointer(a[2 + i], &p[i]))
            return nullptr;
    PyObject *number = PyNumber_Float(a[12]);
    if (number == nullptr)
        return nullptr;
    const double scale = PyFloat_AS_DOUBLE(number);
    Py_DECREF(number);
    if (!pointer(a[13], &p[10]) || !stream(a[14], a[1], &s))
        return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((decode_fn)f)(p[0], p[1], (const uint8_t *)p[2], (const uint8_t *)p[3], (const int32_t *)p[4], p[5], p[6], p[7], p[8],
                        (const int32_t *)p[9], (float)scale, (float *)p[10], s);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// append(function address, current-stream callable, <the 10 arguments of pq_encode_append>)
PyObject *append(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    void *f, *p[10], *s;
    uint64_t n_new;
    if (!count(n, 12) || !pointer(a[0], &f) || !handle(a[2], &p[0]) || !integer(a[5], &n_new))
        return nullptr;
    for (int i = 1; i < 9; ++i)  // new_k, new_v, (n_new), k_codebook, v_codebook, k_codes, v_codes, ctx_len
        if (i != 3 && !pointer(a[2 + i], &p[i]))
            return nullptr;
    if (!stream(a[11], a[1], &s))
        return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((append_fn)f)(p[0], p[1], p[2], (int32_t)(uint32_t)n_new, p[4], p[5], (uint8_t *)p[6], (uint8_t *)p[7],
                        (int32_t *)p[8], s);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {{"decode", (PyCFunction)(void (*)(void))decode, METH_FASTCALL, nullptr},
                         {"append", (PyCFunction)(void (*)(void))append, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pq_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pq_calls(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_value = PyUnicode_InternFromString("value");
    if (s_data_ptr == nullptr || s_cuda_stream == nullptr || s_value == nullptr)
        return nullptr;
    return PyModule_Create(&module);
}
