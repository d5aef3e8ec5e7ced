/* The calls that a training loop makes once per step, for Python: the arguments of zi_grad_norm, zi_grad_norm_noalloc and
 * zi_adamw_step are taken out of their objects here.  On a short tensor such a call is bound by the host, and ctypes
 * spends on its arguments what the library spends on the launch: norm and step on 1003 elements 9.5 us through ctypes, 7.0
 * without any binding.
 *
 * Only the usual forms are taken: a list made by make_tensors (or any ctypes array of zi_tensor with its length), a
 * zi_adamw_config, numbers that are Python's own int and float, addresses as int, None or an object with data_ptr(), a
 * stream as int, None or an object with cuda_stream.  For anything else, and for whatever raises on the way, a function
 * here returns None and the caller goes the general way, which accepts and refuses as it always has.  The GIL is released
 * during the call as ctypes does it. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "zi.h"

static zi_status (*grad_norm)(const zi_tensor*, int32_t, zi_lp_dtype, float, zi_norm_result*, void*, size_t, void*);
static zi_status (*grad_norm_noalloc)(const zi_tensor*, int32_t, zi_lp_dtype, float, zi_norm_result*, void*);
static zi_status (*adamw_step)(const zi_tensor*, int32_t, zi_lp_dtype, const zi_adamw_config*, const zi_norm_result*, void*);
static PyObject *s_data_ptr, *s_cuda_stream, *s_numel, *s_element_size;
static char tensor_format[256], config_format[256];     /* how ctypes describes the two structures */

/* 1 and the value, or 0 without an error set. */
static int as_int(PyObject* x, long long lo, long long hi, long long* out)
{
    int over = 0;
    if (!PyLong_CheckExact(x)) return 0;
    *out = PyLong_AsLongLongAndOverflow(x, &over);
    return !over && *out >= lo && *out <= hi;
}
static int as_float(PyObject* x, float* out)
{
    if (!PyFloat_CheckExact(x)) return 0;
    *out = (float)PyFloat_AS_DOUBLE(x);
    return 1;
}
static int as_pointer(PyObject* x, PyObject* method, PyObject* attribute, void** out)
{
    if (x == Py_None) {
        *out = NULL;
        return 1;
    }
    if (PyLong_CheckExact(x)) {
        Py_INCREF(x);
    } else {
        x = method ? PyObject_CallMethodNoArgs(x, method) : PyObject_GetAttr(x, attribute);
        if (!x) goto no;
        if (!PyLong_CheckExact(x)) goto drop;
    }
    *out = (void*)PyLong_AsUnsignedLongLong(x);
    if (PyErr_Occurred()) goto drop;
    Py_DECREF(x);
    return 1;
drop:
    Py_DECREF(x);
no:
    PyErr_Clear();
    return 0;
}
static int view_of(PyObject* x, const char* format, Py_buffer* view)
{
    if (PyObject_GetBuffer(x, view, PyBUF_FORMAT | PyBUF_ND | PyBUF_WRITABLE) != 0) {
        PyErr_Clear();
        return 0;
    }
    if (view->format && strcmp(view->format, format) == 0) return 1;
    PyBuffer_Release(view);
    return 0;
}
/* The pair (array, length) of make_tensors. */
static int tensors_of(PyObject* x, Py_buffer* view, long long* n)
{
    if (!PyTuple_CheckExact(x) || PyTuple_GET_SIZE(x) != 2) return 0;
    if (!as_int(PyTuple_GET_ITEM(x, 1), INT32_MIN, INT32_MAX, n)) return 0;
    if (!view_of(PyTuple_GET_ITEM(x, 0), tensor_format, view)) return 0;
    if (view->ndim == 1) return 1;
    PyBuffer_Release(view);
    return 0;
}

static PyObject* call_grad_norm(PyObject* self, PyObject* const* a, Py_ssize_t n_args)
{
    long long n, dt, bytes;
    float scale;
    void *out, *ws, *stream;
    Py_buffer list;
    zi_status st;
    if (n_args != 7 || !as_int(a[1], INT32_MIN, INT32_MAX, &dt) || !as_float(a[2], &scale) || !as_pointer(a[3], s_data_ptr, NULL, &out) ||
        !as_pointer(a[4], s_data_ptr, NULL, &ws) || !as_pointer(a[6], NULL, s_cuda_stream, &stream))
        Py_RETURN_NONE;
    if (a[5] == Py_None) {
        PyObject* count = PyObject_CallMethodNoArgs(a[4], s_numel);
        PyObject* size = count ? PyObject_CallMethodNoArgs(a[4], s_element_size) : NULL;
        long long c = 0, s = 0;
        const int ok = count && size && as_int(count, 0, (long long)1 << 40, &c) && as_int(size, 1, 64, &s);
        Py_XDECREF(count);
        Py_XDECREF(size);
        PyErr_Clear();
        if (!ok) Py_RETURN_NONE;
        bytes = c * s;
    } else if (!as_int(a[5], 0, INT64_MAX, &bytes)) {
        Py_RETURN_NONE;
    }
    if (!tensors_of(a[0], &list, &n)) Py_RETURN_NONE;
    Py_BEGIN_ALLOW_THREADS
    st = grad_norm((const zi_tensor*)list.buf, (int32_t)n, (zi_lp_dtype)dt, scale, (zi_norm_result*)out, ws, (size_t)bytes, stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&list);
    return PyLong_FromLong((long)st);
}

static PyObject* call_grad_norm_noalloc(PyObject* self, PyObject* const* a, Py_ssize_t n_args)
{
    long long n, dt;
    float scale;
    void *out, *stream;
    Py_buffer list;
    zi_status st;
    if (n_args != 5 || !as_int(a[1], INT32_MIN, INT32_MAX, &dt) || !as_float(a[2], &scale) || !as_pointer(a[3], s_data_ptr, NULL, &out) ||
        !as_pointer(a[4], NULL, s_cuda_stream, &stream) || !tensors_of(a[0], &list, &n))
        Py_RETURN_NONE;
    Py_BEGIN_ALLOW_THREADS
    st = grad_norm_noalloc((const zi_tensor*)list.buf, (int32_t)n, (zi_lp_dtype)dt, scale, (zi_norm_result*)out, stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&list);
    return PyLong_FromLong((long)st);
}

static PyObject* call_adamw_step(PyObject* self, PyObject* const* a, Py_ssize_t n_args)
{
    long long n, dt;
    void *norm, *stream;
    Py_buffer list, cfg;
    zi_status st;
    if (n_args != 5 || !as_int(a[1], INT32_MIN, INT32_MAX, &dt) || !as_pointer(a[3], s_data_ptr, NULL, &norm) ||
        !as_pointer(a[4], NULL, s_cuda_stream, &stream) || !view_of(a[2], config_format, &cfg))
        Py_RETURN_NONE;
    if (cfg.ndim != 0 || !tensors_of(a[0], &list, &n)) {
        PyBuffer_Release(&cfg);
        Py_RETURN_NONE;
    }
    Py_BEGIN_ALLOW_THREADS
    st = adamw_step((const zi_tensor*)list.buf, (int32_t)n, (zi_lp_dtype)dt, (const zi_adamw_config*)cfg.buf, (const zi_norm_result*)norm, stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&list);
    PyBuffer_Release(&cfg);
    return PyLong_FromLong((long)st);
}

/* bind(address of zi_grad_norm, of zi_grad_norm_noalloc, of zi_adamw_step, a zi_tensor, a zi_adamw_config): True if these
 * are the structures that this module was compiled with. */
static PyObject* bind(PyObject* self, PyObject* const* a, Py_ssize_t n_args)
{
    void* f[3];
    Py_buffer view;
    char* const formats[2] = {tensor_format, config_format};
    const Py_ssize_t sizes[2] = {(Py_ssize_t)sizeof(zi_tensor), (Py_ssize_t)sizeof(zi_adamw_config)};
    int ok = n_args == 5;
    for (int i = 0; ok && i < 3; ++i) ok = as_pointer(a[i], s_data_ptr, NULL, &f[i]) && f[i];
    for (int i = 0; ok && i < 2; ++i) {
        if (PyObject_GetBuffer(a[3 + i], &view, PyBUF_FORMAT | PyBUF_ND) != 0) return NULL;
        ok = view.itemsize == sizes[i] && view.format && strlen(view.format) < sizeof tensor_format;
        if (ok) strcpy(formats[i], view.format);
        PyBuffer_Release(&view);
    }
    if (!ok) Py_RETURN_FALSE;
    grad_norm = (zi_status(*)(const zi_tensor*, int32_t, zi_lp_dtype, float, zi_norm_result*, void*, size_t, void*))f[0];
    grad_norm_noalloc = (zi_status(*)(const zi_tensor*, int32_t, zi_lp_dtype, float, zi_norm_result*, void*))f[1];
    adamw_step = (zi_status(*)(const zi_tensor*, int32_t, zi_lp_dtype, const zi_adamw_config*, const zi_norm_result*, void*))f[2];
    Py_RETURN_TRUE;
}

static PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, NULL},
    {"grad_norm", (PyCFunction)(void (*)(void))call_grad_norm, METH_FASTCALL, NULL},
    {"grad_norm_noalloc", (PyCFunction)(void (*)(void))call_grad_norm_noalloc, METH_FASTCALL, NULL},
    {"adamw_step", (PyCFunction)(void (*)(void))call_adamw_step, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_zi_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__zi_call(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    if (!s_data_ptr || !s_cuda_stream || !s_numel || !s_element_size) return NULL;
    return PyModule_Create(&module);
}
