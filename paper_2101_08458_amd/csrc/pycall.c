/* The calls of an inference loop from Python: the argument conversions of unit.py's launching entry points, natively.
 *
 * A one-launch call spends 2.5 us in the runtime's launch and spent 1.8 us in the conversions of ctypes and the helpers around it
 * (classifier of a batch-1 network, 1x1000x2048 int8, whole call: 4.9 us through ctypes, 3.8 here).  entry(kind, address, types) makes
 * a function of the C entry point at `address` (of the library that unit.py has loaded; this module is not linked to it).  It
 * converts what such a loop passes -- ints, tensors, None, streams, the descriptor structures -- and returns the status, or None for
 * anything else (ints beyond the C type, floats, other structures): the caller then takes the ctypes path, which accepts or refuses it.  The GIL is released around the call, as ctypes does. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <pthread.h>
#include <stdint.h>

static PyObject *s_data_ptr, *s_numel, *s_element_size, *s_cuda_stream;
static PyObject *g_get_device, *g_raw_stream;      /* torch's current device, and the handle of its current stream there */
static volatile int g_streams;                     /* both may be called: torch is initialised, and this is not a forked child */

enum { CONVERTED = 0, OTHER = 1, FAILED = -1 };

static int to_int(PyObject *o, int64_t lo, int64_t hi, int64_t *out)
{
    int overflow = 0;
    if (!PyLong_Check(o)) return OTHER;
    *out = PyLong_AsLongLongAndOverflow(o, &overflow);
    return (overflow || *out < lo || *out > hi) ? OTHER : CONVERTED;
}

static int method_int(PyObject *o, PyObject *name, uint64_t *out)
{
    PyObject *r = PyObject_CallMethodNoArgs(o, name);
    if (!r) return FAILED;
    *out = PyLong_AsUnsignedLongLong(r);
    Py_DECREF(r);
    return (*out == (uint64_t)-1 && PyErr_Occurred()) ? FAILED : CONVERTED;
}

/* device address: of a tensor, or as it is; None is NULL */
static int to_ptr(PyObject *o, void **out)
{
    uint64_t v = 0;
    *out = NULL;
    if (o == Py_None) return CONVERTED;
    if (PyLong_Check(o)) {
        int64_t at;
        if (to_int(o, 0, INT64_MAX, &at)) return OTHER;
        *out = (void *)(uintptr_t)at;
        return CONVERTED;
    }
    const int rc = method_int(o, s_data_ptr, &v);
    *out = (void *)(uintptr_t)v;
    return rc;
}

static int to_ws(PyObject *o, void **ptr, size_t *bytes)
{
    uint64_t p = 0, n = 0, e = 0;
    *ptr = NULL;
    *bytes = 0;
    if (o == Py_None) return CONVERTED;
    if (method_int(o, s_data_ptr, &p) || method_int(o, s_numel, &n) || method_int(o, s_element_size, &e)) return FAILED;
    *ptr = (void *)(uintptr_t)p;
    *bytes = (size_t)(n * e);
    return CONVERTED;
}

/* address of a ctypes structure of exactly the given type (it lives as long as the caller's reference) */
static int to_struct(PyObject *o, PyObject *type, void **out)
{
    Py_buffer view;
    if ((PyObject *)Py_TYPE(o) != type) return OTHER;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE)) return FAILED;
    *out = view.buf;
    PyBuffer_Release(&view);
    return CONVERTED;
}

static int to_stream(PyObject *o, void **out)
{
    if (o != Py_None) {
        if (PyLong_Check(o)) return to_ptr(o, out);
        PyObject *h = PyObject_GetAttr(o, s_cuda_stream);
        if (!h) return FAILED;
        const int rc = PyLong_Check(h) ? to_ptr(h, out) : OTHER;
        Py_DECREF(h);
        return rc;
    }
    if (!g_streams) return OTHER;
    PyObject *dev = PyObject_CallNoArgs(g_get_device);
    if (!dev) return FAILED;
    PyObject *r = PyObject_CallOneArg(g_raw_stream, dev);
    Py_DECREF(dev);
    if (!r) return FAILED;
    *out = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return (!*out && PyErr_Occurred()) ? FAILED : CONVERTED;
}

/* what an entry function carries: the address of the C function, and the structure types it takes */
typedef struct { void *fn; PyObject *desc, *requant; } entry_t;
static entry_t *carried(PyObject *self) { return (entry_t *)PyCapsule_GetPointer(self, "unit entry"); }

#define TRY(call) do { const int rc_ = (call); if (rc_ == FAILED) return NULL; if (rc_ == OTHER) Py_RETURN_NONE; } while (0)
#define CALL(expr) do { int st_; Py_BEGIN_ALLOW_THREADS st_ = (expr); Py_END_ALLOW_THREADS return PyLong_FromLong(st_); } while (0)
#define ARGS(n) do { if (nargs != (n)) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return NULL; } } while (0)

static int opt_requant(entry_t *e, PyObject *o, void **out)
{
    *out = NULL;
    return o == Py_None ? CONVERTED : to_struct(o, e->requant, out);
}

/* m, n, k, A, lda, B, ldb, C, ldc, ws, stream */
static PyObject *call_matmul(PyObject *self, PyObject *const *a, Py_ssize_t nargs)
{
    typedef int (*fn_t)(int32_t, int32_t, int32_t, const void *, int64_t, const void *, int64_t, void *, int64_t, void *, size_t, void *);
    entry_t *e = carried(self);
    int64_t m, n, k, lda, ldb, ldc;
    void *A, *B, *C, *ws, *st;
    size_t wb;
    ARGS(11);
    TRY(to_int(a[0], INT32_MIN, INT32_MAX, &m));  TRY(to_int(a[1], INT32_MIN, INT32_MAX, &n));  TRY(to_int(a[2], INT32_MIN, INT32_MAX, &k));
    TRY(to_int(a[4], INT64_MIN, INT64_MAX, &lda));  TRY(to_int(a[6], INT64_MIN, INT64_MAX, &ldb));  TRY(to_int(a[8], INT64_MIN, INT64_MAX, &ldc));
    TRY(to_ptr(a[3], &A));  TRY(to_ptr(a[5], &B));  TRY(to_ptr(a[7], &C));  TRY(to_ws(a[9], &ws, &wb));  TRY(to_stream(a[10], &st));
    CALL(((fn_t)e->fn)((int32_t)m, (int32_t)n, (int32_t)k, A, lda, B, ldb, C, ldc, ws, wb, st));
}

/* d, x, w, y, ws, stream */
static PyObject *call_conv(PyObject *self, PyObject *const *a, Py_ssize_t nargs)
{
    typedef int (*fn_t)(const void *, const void *, const void *, void *, void *, size_t, void *);
    entry_t *e = carried(self);
    void *d, *x, *w, *y, *ws, *st;
    size_t wb;
    ARGS(6);
    TRY(to_struct(a[0], e->desc, &d));  TRY(to_ptr(a[1], &x));  TRY(to_ptr(a[2], &w));  TRY(to_ptr(a[3], &y));
    TRY(to_ws(a[4], &ws, &wb));  TRY(to_stream(a[5], &st));
    CALL(((fn_t)e->fn)(d, x, w, y, ws, wb, st));
}

/* d, x, w, y_i32, rq, y_i8, ws, stream */
static PyObject *call_conv_i8(PyObject *self, PyObject *const *a, Py_ssize_t nargs)
{
    typedef int (*fn_t)(const void *, const void *, const void *, void *, const void *, void *, void *, size_t, void *);
    entry_t *e = carried(self);
    void *d, *x, *w, *y, *rq, *y8, *ws, *st;
    size_t wb;
    ARGS(8);
    TRY(to_struct(a[0], e->desc, &d));  TRY(to_ptr(a[1], &x));  TRY(to_ptr(a[2], &w));  TRY(to_ptr(a[3], &y));
    TRY(opt_requant(e, a[4], &rq));  TRY(to_ptr(a[5], &y8));  TRY(to_ws(a[6], &ws, &wb));  TRY(to_stream(a[7], &st));
    CALL(((fn_t)e->fn)(d, x, w, y, rq, y8, ws, wb, st));
}

/* d, x_packed, w_packed, y_i32, rq, y_i8, y_packed, ws, stream */
static PyObject *call_packed_i8(PyObject *self, PyObject *const *a, Py_ssize_t nargs)
{
    typedef int (*fn_t)(const void *, const void *, const void *, void *, const void *, void *, void *, void *, size_t, void *);
    entry_t *e = carried(self);
    void *d, *x, *w, *y, *rq, *y8, *yp, *ws, *st;
    size_t wb;
    ARGS(9);
    TRY(to_struct(a[0], e->desc, &d));  TRY(to_ptr(a[1], &x));  TRY(to_ptr(a[2], &w));  TRY(to_ptr(a[3], &y));
    TRY(opt_requant(e, a[4], &rq));  TRY(to_ptr(a[5], &y8));  TRY(to_ptr(a[6], &yp));  TRY(to_ws(a[7], &ws, &wb));  TRY(to_stream(a[8], &st));
    CALL(((fn_t)e->fn)(d, x, w, y, rq, y8, yp, ws, wb, st));
}

static PyMethodDef kinds[] = {
    {"matmul", (PyCFunction)(void (*)(void))call_matmul, METH_FASTCALL, NULL},
    {"conv", (PyCFunction)(void (*)(void))call_conv, METH_FASTCALL, NULL},
    {"conv_i8", (PyCFunction)(void (*)(void))call_conv_i8, METH_FASTCALL, NULL},
    {"packed_i8", (PyCFunction)(void (*)(void))call_packed_i8, METH_FASTCALL, NULL},
};

static void free_entry(PyObject *capsule)
{
    entry_t *e = carried(capsule);
    Py_XDECREF(e->desc);
    Py_XDECREF(e->requant);
    PyMem_Free(e);
}

/* entry(kind, address, descriptor type or None, requantise type or None) */
static PyObject *make_entry(PyObject *self, PyObject *args)
{
    const char *kind;
    PyObject *addr, *desc, *requant;
    (void)self;
    if (!PyArg_ParseTuple(args, "sOOO", &kind, &addr, &desc, &requant)) return NULL;
    void *fn = PyLong_AsVoidPtr(addr);
    if (!fn) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no function address");
        return NULL;
    }
    for (size_t i = 0; i < sizeof kinds / sizeof kinds[0]; ++i) {
        if (strcmp(kinds[i].ml_name, kind)) continue;
        entry_t *e = (entry_t *)PyMem_Malloc(sizeof *e);
        if (!e) return PyErr_NoMemory();
        Py_INCREF(desc);
        Py_INCREF(requant);
        e->fn = fn;
        e->desc = desc;
        e->requant = requant;
        PyObject *capsule = PyCapsule_New(e, "unit entry", free_entry);
        if (!capsule) {
            Py_DECREF(desc);
            Py_DECREF(requant);
            PyMem_Free(e);
            return NULL;
        }
        PyObject *f = PyCFunction_NewEx(&kinds[i], capsule, NULL);
        Py_DECREF(capsule);
        return f;
    }
    PyErr_Format(PyExc_ValueError, "no entry of kind %s", kind);
    return NULL;
}

/* streams(get_device, raw_stream): from now on a call without a stream asks these; torch is initialised in this process */
static PyObject *set_streams(PyObject *self, PyObject *args)
{
    PyObject *dev, *raw;
    (void)self;
    if (!PyArg_ParseTuple(args, "OO", &dev, &raw)) return NULL;
    Py_INCREF(dev);
    Py_INCREF(raw);
    Py_XSETREF(g_get_device, dev);
    Py_XSETREF(g_raw_stream, raw);
    g_streams = 1;
    Py_RETURN_NONE;
}

/* a forked child has no device: torch's own call refuses there */
static void in_child(void) { g_streams = 0; }

static PyMethodDef methods[] = {
    {"entry", make_entry, METH_VARARGS, NULL},
    {"streams", set_streams, METH_VARARGS, NULL},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_unitcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__unitcall(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!s_data_ptr || !s_numel || !s_element_size || !s_cuda_stream || pthread_atfork(NULL, NULL, in_child)) return NULL;
    return PyModule_Create(&module);
}
