/* Argument marshalling of the calls a training step makes, as a CPython extension: None is NULL, an int is an address or a number, a tensor is
 * asked for its data_ptr(); at a fifth of the time that ctypes and the helpers in cgbn.py take for the same (a step of a small layer is
 * host bound: of 9 us a call they took 4).  Whatever is not so plain (a ctypes object, a wrong type, a name that is not in the table) is
 * answered NotImplemented before anything is called, and cgbn.py takes the call through ctypes, which accepts or refuses it.  The library is not
 * linked: bind() is handed the addresses of its functions by whoever loaded it. */

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "cgbn.h"

typedef cgbn_status (*forward_fn)(const void*, int, int, int, int, cgbn_layout, int, const float*, const float*, float, void*, float*, float*,
                                  cgbn_dtype, float*, void*, size_t, void*);
typedef cgbn_status (*forward_relu_fn)(const void*, const void*, int, int, int, int, cgbn_layout, int, const float*, const float*, float, void*,
                                       float*, float*, cgbn_dtype, float*, void*, size_t, void*);
typedef cgbn_status (*backward_fn)(const void*, const void*, const float*, const float*, const float*, void*, float*, float*, int, int, int, int,
                                   cgbn_layout, int, cgbn_dtype, const float*, void*, size_t, void*);
typedef cgbn_status (*backward_relu_fn)(const void*, const void*, const void*, const float*, const float*, const float*, void*, void*, float*,
                                        float*, int, int, int, int, cgbn_layout, int, cgbn_dtype, const float*, void*, size_t, void*);
typedef cgbn_status (*frozen_forward_fn)(const void*, int, int, int, int, cgbn_layout, cgbn_dtype, const float*, const float*, const float*,
                                         const float*, float, void*, void*);
typedef cgbn_status (*frozen_backward_fn)(const void*, int, int, int, int, cgbn_layout, cgbn_dtype, const float*, const float*, float, void*,
                                          void*);

static forward_fn g_forward;
static forward_relu_fn g_forward_relu;
static backward_fn g_backward;
static backward_relu_fn g_backward_relu;
static frozen_forward_fn g_frozen_forward;
static frozen_backward_fn g_frozen_backward;
static PyObject *g_layouts, *g_dtypes, *g_stream;       /* name -> number; () -> the current stream's address */
static PyObject *g_data_ptr, *g_numel, *g_element_size;

/* Converters: each returns 0 and clears *plain for what ctypes has to deal with, and does nothing once *plain is 0. */
static unsigned long long number(PyObject* o, int* plain)
{
    if (*plain && PyLong_Check(o)) return PyLong_AsUnsignedLongLongMask(o);
    *plain = 0;
    return 0;
}
/* the number that a method without arguments returns */
static unsigned long long asked(PyObject* o, PyObject* method, int* plain)
{
    unsigned long long v;
    PyObject* a = PyObject_CallMethodNoArgs(o, method);
    if (!a) { *plain = 0; return 0; }
    v = number(a, plain);
    Py_DECREF(a);
    return v;
}
static void* ptr(PyObject* o, int* plain)
{
    if (!*plain || o == Py_None) return NULL;
    return (void*)(uintptr_t)(PyLong_Check(o) ? number(o, plain) : asked(o, g_data_ptr, plain));
}
static int num(PyObject* o, int* plain)
{
    return (int)number(o, plain);
}
static int name(PyObject* table, PyObject* o, int* plain)
{
    if (*plain && PyUnicode_Check(o)) {
        o = PyDict_GetItemWithError(table, o);        /* borrowed */
        if (!o) { *plain = 0; return 0; }
    }
    return (int)number(o, plain);
}
static float real(PyObject* o, int* plain)
{
    if (*plain && PyFloat_Check(o)) return (float)PyFloat_AS_DOUBLE(o);
    *plain = 0;
    return 0.f;
}
/* the workspace's size: what the caller says, else the tensor's own */
static size_t room(PyObject* workspace, PyObject* bytes, int* plain)
{
    unsigned long long n;
    if (!*plain) return 0;
    if (bytes != Py_None) return (size_t)number(bytes, plain);
    if (workspace == Py_None) return 0;
    n = asked(workspace, g_numel, plain);
    return *plain ? (size_t)(n * asked(workspace, g_element_size, plain)) : 0;
}
static void* stream(PyObject* o, int* plain)
{
    void* v;
    PyObject* a;
    if (!*plain) return NULL;
    if (PyLong_Check(o)) return (void*)(uintptr_t)number(o, plain);
    a = PyObject_CallOneArg(g_stream, o);
    if (!a) { *plain = 0; return NULL; }
    v = a == Py_None ? NULL : (void*)(uintptr_t)number(a, plain);
    Py_DECREF(a);
    return v;
}

#define ARGS(count_)                                                                                     \
    int plain = 1;                                                                                       \
    if (n != (count_)) { PyErr_Format(PyExc_TypeError, "%d arguments, %zd given", (count_), n); return NULL; } \
    if (!g_forward) { PyErr_SetString(PyExc_RuntimeError, "bind() first"); return NULL; }
/* (the launch may wait for room in a queue) */
#define CALL(call_)                                                                                      \
    do {                                                                                                 \
        cgbn_status s_;                                                                                  \
        if (!plain) {                                                                                    \
            if (PyErr_Occurred()) {                                                                      \
                if (!PyErr_ExceptionMatches(PyExc_Exception)) return NULL;       /* an interrupt */      \
                PyErr_Clear();                                                                           \
            }                                                                                            \
            Py_RETURN_NOTIMPLEMENTED;                                                                    \
        }                                                                                                \
        Py_BEGIN_ALLOW_THREADS                                                                           \
        s_ = (call_);                                                                                    \
        Py_END_ALLOW_THREADS                                                                             \
        return PyLong_FromLong((long)s_);                                                                \
    } while (0)

static PyObject* forward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(18)
    const void* x = ptr(a[0], &plain);
    const int N = num(a[1], &plain), C = num(a[2], &plain), H = num(a[3], &plain), W = num(a[4], &plain), layout = name(g_layouts, a[5], &plain), K = num(a[6], &plain);
    const float *gamma = ptr(a[7], &plain), *beta = ptr(a[8], &plain);
    const float eps = real(a[9], &plain);
    void* y = ptr(a[10], &plain);
    float *mean = ptr(a[11], &plain), *invstd = ptr(a[12], &plain);
    const int dtype = name(g_dtypes, a[13], &plain);
    float* mean_lo = ptr(a[14], &plain);
    void* ws = ptr(a[15], &plain);
    const size_t bytes = room(a[15], a[16], &plain);
    void* st = stream(a[17], &plain);
    CALL(g_forward(x, N, C, H, W, layout, K, gamma, beta, eps, y, mean, invstd, dtype, mean_lo, ws, bytes, st));
}
static PyObject* forward_relu(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(19)
    const void *x = ptr(a[0], &plain), *shortcut = ptr(a[1], &plain);
    const int N = num(a[2], &plain), C = num(a[3], &plain), H = num(a[4], &plain), W = num(a[5], &plain), layout = name(g_layouts, a[6], &plain), K = num(a[7], &plain);
    const float *gamma = ptr(a[8], &plain), *beta = ptr(a[9], &plain);
    const float eps = real(a[10], &plain);
    void* y = ptr(a[11], &plain);
    float *mean = ptr(a[12], &plain), *invstd = ptr(a[13], &plain);
    const int dtype = name(g_dtypes, a[14], &plain);
    float* mean_lo = ptr(a[15], &plain);
    void* ws = ptr(a[16], &plain);
    const size_t bytes = room(a[16], a[17], &plain);
    void* st = stream(a[18], &plain);
    CALL(g_forward_relu(x, shortcut, N, C, H, W, layout, K, gamma, beta, eps, y, mean, invstd, dtype, mean_lo, ws, bytes, st));
}
static PyObject* backward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(19)
    const void *dy = ptr(a[0], &plain), *x = ptr(a[1], &plain);
    const float *mean = ptr(a[2], &plain), *invstd = ptr(a[3], &plain), *gamma = ptr(a[4], &plain);
    void* dx = ptr(a[5], &plain);
    float *dgamma = ptr(a[6], &plain), *dbeta = ptr(a[7], &plain);
    const int N = num(a[8], &plain), C = num(a[9], &plain), H = num(a[10], &plain), W = num(a[11], &plain), layout = name(g_layouts, a[12], &plain), K = num(a[13], &plain);
    const int dtype = name(g_dtypes, a[14], &plain);
    const float* mean_lo = ptr(a[15], &plain);
    void* ws = ptr(a[16], &plain);
    const size_t bytes = room(a[16], a[17], &plain);
    void* st = stream(a[18], &plain);
    CALL(g_backward(dy, x, mean, invstd, gamma, dx, dgamma, dbeta, N, C, H, W, layout, K, dtype, mean_lo, ws, bytes, st));
}
static PyObject* backward_relu(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(21)
    const void *dy = ptr(a[0], &plain), *y = ptr(a[1], &plain), *x = ptr(a[2], &plain);
    const float *mean = ptr(a[3], &plain), *invstd = ptr(a[4], &plain), *gamma = ptr(a[5], &plain);
    void *dx = ptr(a[6], &plain), *dshortcut = ptr(a[7], &plain);
    float *dgamma = ptr(a[8], &plain), *dbeta = ptr(a[9], &plain);
    const int N = num(a[10], &plain), C = num(a[11], &plain), H = num(a[12], &plain), W = num(a[13], &plain), layout = name(g_layouts, a[14], &plain), K = num(a[15], &plain);
    const int dtype = name(g_dtypes, a[16], &plain);
    const float* mean_lo = ptr(a[17], &plain);
    void* ws = ptr(a[18], &plain);
    const size_t bytes = room(a[18], a[19], &plain);
    void* st = stream(a[20], &plain);
    CALL(g_backward_relu(dy, y, x, mean, invstd, gamma, dx, dshortcut, dgamma, dbeta, N, C, H, W, layout, K, dtype, mean_lo, ws, bytes, st));
}
static PyObject* frozen_forward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(14)
    const void* x = ptr(a[0], &plain);
    const int N = num(a[1], &plain), C = num(a[2], &plain), H = num(a[3], &plain), W = num(a[4], &plain), layout = name(g_layouts, a[5], &plain), dtype = name(g_dtypes, a[6], &plain);
    const float *fixed_mean = ptr(a[7], &plain), *fixed_var = ptr(a[8], &plain), *gamma = ptr(a[9], &plain), *beta = ptr(a[10], &plain);
    const float eps = real(a[11], &plain);
    void* y = ptr(a[12], &plain);
    void* st = stream(a[13], &plain);
    CALL(g_frozen_forward(x, N, C, H, W, layout, dtype, fixed_mean, fixed_var, gamma, beta, eps, y, st));
}
static PyObject* frozen_backward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(12)
    const void* dy = ptr(a[0], &plain);
    const int N = num(a[1], &plain), C = num(a[2], &plain), H = num(a[3], &plain), W = num(a[4], &plain), layout = name(g_layouts, a[5], &plain), dtype = name(g_dtypes, a[6], &plain);
    const float *fixed_var = ptr(a[7], &plain), *gamma = ptr(a[8], &plain);
    const float eps = real(a[9], &plain);
    void* dx = ptr(a[10], &plain);
    void* st = stream(a[11], &plain);
    CALL(g_frozen_backward(dy, N, C, H, W, layout, dtype, fixed_var, gamma, eps, dx, st));
}

/* bind(addresses of the six functions, layouts, dtypes, stream) */
static PyObject* bind(PyObject* self, PyObject* args)
{
    unsigned long long f[6];
    PyObject *layouts, *dtypes, *st;
    (void)self;
    if (!PyArg_ParseTuple(args, "(KKKKKK)OOO", &f[0], &f[1], &f[2], &f[3], &f[4], &f[5], &layouts, &dtypes, &st)) return NULL;
    Py_INCREF(layouts);
    Py_INCREF(dtypes);
    Py_INCREF(st);
    Py_XSETREF(g_layouts, layouts);
    Py_XSETREF(g_dtypes, dtypes);
    Py_XSETREF(g_stream, st);
    g_forward = (forward_fn)(uintptr_t)f[0];
    g_forward_relu = (forward_relu_fn)(uintptr_t)f[1];
    g_backward = (backward_fn)(uintptr_t)f[2];
    g_backward_relu = (backward_relu_fn)(uintptr_t)f[3];
    g_frozen_forward = (frozen_forward_fn)(uintptr_t)f[4];
    g_frozen_backward = (frozen_backward_fn)(uintptr_t)f[5];
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, NULL},
    {"forward", (PyCFunction)(void (*)(void))forward, METH_FASTCALL, NULL},
    {"forward_relu", (PyCFunction)(void (*)(void))forward_relu, METH_FASTCALL, NULL},
    {"backward", (PyCFunction)(void (*)(void))backward, METH_FASTCALL, NULL},
    {"backward_relu", (PyCFunction)(void (*)(void))backward_relu, METH_FASTCALL, NULL},
    {"frozen_forward", (PyCFunction)(void (*)(void))frozen_forward, METH_FASTCALL, NULL},
    {"frozen_backward", (PyCFunction)(void (*)(void))frozen_backward, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_cgbn_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__cgbn_call(void)
{
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_numel = PyUnicode_InternFromString("numel");
    g_element_size = PyUnicode_InternFromString("element_size");
    if (!g_data_ptr || !g_numel || !g_element_size) return NULL;
    return PyModule_Create(&module);
}
