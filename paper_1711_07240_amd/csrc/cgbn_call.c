/* Argument marshalling of the calls a training step makes, as a CPython extension: the same conversions as ctypes and the helpers in
 * cgbn.py make (None is NULL, a number is an address, anything else is asked for its data_ptr()), at a fifth of the time.  A step of a
 * small layer is host bound: of 9 us a call, ctypes and the helpers took 4.  The library is not linked: bind() is handed
 * the addresses of its functions by whoever loaded it. */

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

/* Converters: each does nothing once an exception is set. */
static void* ptr(PyObject* o)
{
    void* v;
    PyObject *a, *n;
    if (o == Py_None || PyErr_Occurred()) return NULL;
    if (PyLong_Check(o)) return (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    a = PyObject_CallMethodNoArgs(o, g_data_ptr);
    if (!a) return NULL;
    n = PyNumber_Long(a);
    Py_DECREF(a);
    if (!n) return NULL;
    v = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return v;
}
static int num(PyObject* o)
{
    return PyErr_Occurred() ? 0 : (int)PyLong_AsUnsignedLongMask(o);
}
static int name(PyObject* table, PyObject* o)
{
    PyObject* v;
    int r;
    if (PyErr_Occurred()) return 0;
    if (PyUnicode_Check(o)) {
        v = PyObject_GetItem(table, o);       /* KeyError */
    } else {
        v = PyNumber_Long(o);
    }
    if (!v) return 0;
    r = (int)PyLong_AsUnsignedLongMask(v);
    Py_DECREF(v);
    return r;
}
static float real(PyObject* o)
{
    PyObject* f;
    double v;
    if (PyErr_Occurred()) return 0.f;
    f = PyNumber_Float(o);
    if (!f) return 0.f;
    v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)v;
}
/* the workspace's size: what the caller says, else the tensor's own */
static size_t room(PyObject* workspace, PyObject* bytes)
{
    PyObject *a, *b, *c;
    size_t v;
    if (PyErr_Occurred()) return 0;
    if (bytes != Py_None) return (size_t)PyLong_AsUnsignedLongLongMask(bytes);
    if (workspace == Py_None) return 0;
    a = PyObject_CallMethodNoArgs(workspace, g_numel);
    b = a ? PyObject_CallMethodNoArgs(workspace, g_element_size) : NULL;
    c = b ? PyNumber_Multiply(a, b) : NULL;
    Py_XDECREF(a);
    Py_XDECREF(b);
    if (!c) return 0;
    v = (size_t)PyLong_AsUnsignedLongLongMask(c);
    Py_DECREF(c);
    return v;
}
static void* stream(PyObject* o)
{
    PyObject* a;
    void* v;
    if (PyErr_Occurred()) return NULL;
    if (PyLong_Check(o)) return (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    a = PyObject_CallOneArg(g_stream, o);
    if (!a) return NULL;
    v = a == Py_None ? NULL : (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(a);
    Py_DECREF(a);
    return v;
}

#define ARGS(count_)                                                                                     \
    if (n != (count_)) { PyErr_Format(PyExc_TypeError, "%d arguments, %zd given", (count_), n); return NULL; } \
    if (!g_forward) { PyErr_SetString(PyExc_RuntimeError, "bind() first"); return NULL; }
/* (the launch may wait for room in a queue) */
#define CALL(call_)                                                                                      \
    do {                                                                                                 \
        cgbn_status s_;                                                                                  \
        if (PyErr_Occurred()) return NULL;                                                               \
        Py_BEGIN_ALLOW_THREADS                                                                           \
        s_ = (call_);                                                                                    \
        Py_END_ALLOW_THREADS                                                                             \
        return PyLong_FromLong((long)s_);                                                                \
    } while (0)

static PyObject* forward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(18)
    const void* x = ptr(a[0]);
    const int N = num(a[1]), C = num(a[2]), H = num(a[3]), W = num(a[4]), layout = name(g_layouts, a[5]), K = num(a[6]);
    const float *gamma = ptr(a[7]), *beta = ptr(a[8]);
    const float eps = real(a[9]);
    void* y = ptr(a[10]);
    float *mean = ptr(a[11]), *invstd = ptr(a[12]);
    const int dtype = name(g_dtypes, a[13]);
    float* mean_lo = ptr(a[14]);
    void* ws = ptr(a[15]);
    const size_t bytes = room(a[15], a[16]);
    void* st = stream(a[17]);
    CALL(g_forward(x, N, C, H, W, layout, K, gamma, beta, eps, y, mean, invstd, dtype, mean_lo, ws, bytes, st));
}
static PyObject* forward_relu(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(19)
    const void *x = ptr(a[0]), *shortcut = ptr(a[1]);
    const int N = num(a[2]), C = num(a[3]), H = num(a[4]), W = num(a[5]), layout = name(g_layouts, a[6]), K = num(a[7]);
    const float *gamma = ptr(a[8]), *beta = ptr(a[9]);
    const float eps = real(a[10]);
    void* y = ptr(a[11]);
    float *mean = ptr(a[12]), *invstd = ptr(a[13]);
    const int dtype = name(g_dtypes, a[14]);
    float* mean_lo = ptr(a[15]);
    void* ws = ptr(a[16]);
    const size_t bytes = room(a[16], a[17]);
    void* st = stream(a[18]);
    CALL(g_forward_relu(x, shortcut, N, C, H, W, layout, K, gamma, beta, eps, y, mean, invstd, dtype, mean_lo, ws, bytes, st));
}
static PyObject* backward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(19)
    const void *dy = ptr(a[0]), *x = ptr(a[1]);
    const float *mean = ptr(a[2]), *invstd = ptr(a[3]), *gamma = ptr(a[4]);
    void* dx = ptr(a[5]);
    float *dgamma = ptr(a[6]), *dbeta = ptr(a[7]);
    const int N = num(a[8]), C = num(a[9]), H = num(a[10]), W = num(a[11]), layout = name(g_layouts, a[12]), K = num(a[13]);
    const int dtype = name(g_dtypes, a[14]);
    const float* mean_lo = ptr(a[15]);
    void* ws = ptr(a[16]);
    const size_t bytes = room(a[16], a[17]);
    void* st = stream(a[18]);
    CALL(g_backward(dy, x, mean, invstd, gamma, dx, dgamma, dbeta, N, C, H, W, layout, K, dtype, mean_lo, ws, bytes, st));
}
static PyObject* backward_relu(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(21)
    const void *dy = ptr(a[0]), *y = ptr(a[1]), *x = ptr(a[2]);
    const float *mean = ptr(a[3]), *invstd = ptr(a[4]), *gamma = ptr(a[5]);
    void *dx = ptr(a[6]), *dshortcut = ptr(a[7]);
    float *dgamma = ptr(a[8]), *dbeta = ptr(a[9]);
    const int N = num(a[10]), C = num(a[11]), H = num(a[12]), W = num(a[13]), layout = name(g_layouts, a[14]), K = num(a[15]);
    const int dtype = name(g_dtypes, a[16]);
    const float* mean_lo = ptr(a[17]);
    void* ws = ptr(a[18]);
    const size_t bytes = room(a[18], a[19]);
    void* st = stream(a[20]);
    CALL(g_backward_relu(dy, y, x, mean, invstd, gamma, dx, dshortcut, dgamma, dbeta, N, C, H, W, layout, K, dtype, mean_lo, ws, bytes, st));
}
static PyObject* frozen_forward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(14)
    const void* x = ptr(a[0]);
    const int N = num(a[1]), C = num(a[2]), H = num(a[3]), W = num(a[4]), layout = name(g_layouts, a[5]), dtype = name(g_dtypes, a[6]);
    const float *fixed_mean = ptr(a[7]), *fixed_var = ptr(a[8]), *gamma = ptr(a[9]), *beta = ptr(a[10]);
    const float eps = real(a[11]);
    void* y = ptr(a[12]);
    void* st = stream(a[13]);
    CALL(g_frozen_forward(x, N, C, H, W, layout, dtype, fixed_mean, fixed_var, gamma, beta, eps, y, st));
}
static PyObject* frozen_backward(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    ARGS(12)
    const void* dy = ptr(a[0]);
    const int N = num(a[1]), C = num(a[2]), H = num(a[3]), W = num(a[4]), layout = name(g_layouts, a[5]), dtype = name(g_dtypes, a[6]);
    const float *fixed_var = ptr(a[7]), *gamma = ptr(a[8]);
    const float eps = real(a[9]);
    void* dx = ptr(a[10]);
    void* st = stream(a[11]);
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
