/* The calls of a program's inner loop as a CPython module: arguments go from Python ints to the C ABI
 * of libfscnn.so without ctypes, whose conversions cost 4 us a call -- as much as a small layer's
 * launch, and what bounds back-to-back small launches (0.3 us here).  Marshalling only: pointers are
 * ints (None = NULL), checks and allocation stay in fscnn.py, the library is the one it has loaded. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "fscnn.h"

/* entry points of the loaded library, set by bind() */
static struct {
    __typeof__(&fscnn_conv2d_sparse_filter_ex) conv_ex;
    __typeof__(&fscnn_conv2d_sparse_filter_pool2x2) conv_pool;
    __typeof__(&fscnn_conv2d_sparse_filter_leaky) conv_leaky;
    __typeof__(&fscnn_conv2d_sparse_filter_emit) emit;
    __typeof__(&fscnn_conv2d_sparse_filter_emit_into) emit_into;
    __typeof__(&fscnn_conv2d_sparse_input) conv_si;
    __typeof__(&fscnn_conv2d_sparse_input_prepared) conv_sip;
    __typeof__(&fscnn_filter_compress) filter_compress;
    __typeof__(&fscnn_filter_info) filter_info;
    __typeof__(&fscnn_input_compress) input_compress;
    __typeof__(&fscnn_input_info) input_info;
    __typeof__(&fscnn_sparse_transpose) transpose;
    __typeof__(&fscnn_sparse_tensor_transpose) tensor_transpose;
} L;

static const char *const kNames[] = {
    "fscnn_conv2d_sparse_filter_ex", "fscnn_conv2d_sparse_filter_pool2x2", "fscnn_conv2d_sparse_filter_leaky",
    "fscnn_conv2d_sparse_filter_emit", "fscnn_conv2d_sparse_filter_emit_into", "fscnn_conv2d_sparse_input",
    "fscnn_conv2d_sparse_input_prepared", "fscnn_filter_compress", "fscnn_filter_info", "fscnn_input_compress",
    "fscnn_input_info", "fscnn_sparse_transpose", "fscnn_sparse_tensor_transpose",
};
enum { kEntries = sizeof(kNames) / sizeof(kNames[0]) };
_Static_assert(sizeof(L) == kEntries * sizeof(void *), "one name per entry point");

/* Argument readers: a failed conversion sets *bad and leaves the Python error for the caller. */
static int geti(PyObject *o, int *bad)
{
    long v;
    if (PyLong_Check(o)) {
        v = PyLong_AsLong(o);
    } else {   /* any other number by its integer value, as int() takes it (which refuses infinities and NaN) */
        PyObject *n = PyNumber_Long(o);
        v = n ? PyLong_AsLong(n) : -1;
        Py_XDECREF(n);
    }
    if (v == -1 && PyErr_Occurred()) *bad = 1;
    else if (v != (int)v) {
        PyErr_SetString(PyExc_OverflowError, "argument does not fit an int");
        *bad = 1;
    }
    return (int)v;
}
static void *getp(PyObject *o, int *bad)
{
    if (o == Py_None) return NULL;
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) *bad = 1;
    return p;
}
static int wrong_count(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want) return 0;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd wanted", n, want);
    return 1;
}
#define CALL(expr)                          \
    do {                                    \
        if (bad || !L.conv_ex) {            \
            if (!bad) PyErr_SetString(PyExc_RuntimeError, "bind() first"); \
            return NULL;                    \
        }                                   \
        Py_BEGIN_ALLOW_THREADS st = (expr); \
        Py_END_ALLOW_THREADS                \
    } while (0)

/* bind({name: address}) */
static PyObject *py_bind(PyObject *self, PyObject *map)
{
    void *p[kEntries];
    for (int i = 0; i < kEntries; ++i) {
        PyObject *v = PyDict_GetItemString(map, kNames[i]);
        p[i] = v ? PyLong_AsVoidPtr(v) : NULL;
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "%s", kNames[i]);
            return NULL;
        }
    }
    memcpy(&L, p, sizeof(L));
    Py_RETURN_NONE;
}

/* conv(kind, f, x, N, C, H, W, sh, sw, ph, pw, bias, act, y, x_layout, y_layout, variant, stream) -> status
 * kind 0: act = relu; 1: merged pool, act = relu; 2: act = negative slope */
static PyObject *py_conv(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    if (wrong_count(n, 18)) return NULL;
    int bad = 0, v[8], st = 0;
    const int kind = geti(a[0], &bad);
    void *f = getp(a[1], &bad), *x = getp(a[2], &bad);
    for (int i = 0; i < 8; ++i) v[i] = geti(a[3 + i], &bad);
    void *b = getp(a[11], &bad);
    float slope = 0.0f;
    int relu = 0;
    if (kind == 2) {
        const double d = PyFloat_AsDouble(a[12]);
        if (d == -1.0 && PyErr_Occurred()) bad = 1;
        slope = (float)d;
    } else {
        relu = geti(a[12], &bad);
    }
    void *y = getp(a[13], &bad);
    const int xl = geti(a[14], &bad), yl = geti(a[15], &bad), var = geti(a[16], &bad);
    void *s = getp(a[17], &bad);
    CALL(kind == 2   ? L.conv_leaky(f, x, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], b, slope, y, xl, yl, var, s)
         : kind == 1 ? L.conv_pool(f, x, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], b, relu, y, xl, yl, var, s)
                     : L.conv_ex(f, x, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], b, relu, y, xl, yl, var, s));
    return PyLong_FromLong(st);
}

/* emit(f, x, N, C, H, W, sh, sw, ph, pw, bias, relu, y, stream, into) -> (status, handle); into: None or a handle */
static PyObject *py_emit(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    if (wrong_count(n, 15)) return NULL;
    int bad = 0, v[8], st = 0;
    void *f = getp(a[0], &bad), *x = getp(a[1], &bad);
    for (int i = 0; i < 8; ++i) v[i] = geti(a[2 + i], &bad);
    void *b = getp(a[10], &bad);
    const int relu = geti(a[11], &bad);
    void *y = getp(a[12], &bad), *s = getp(a[13], &bad);
    fscnn_input_t *h = getp(a[14], &bad);
    CALL(h ? L.emit_into(f, x, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], b, relu, y, s, h)
           : L.emit(f, x, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], b, relu, y, s, &h));
    return Py_BuildValue("iN", st, PyLong_FromVoidPtr(h));
}

/* conv_si(in, w, K, R, S, sh, sw, ph, pw, bias, relu, y, stream) -> status */
static PyObject *py_conv_si(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    if (wrong_count(n, 13)) return NULL;
    int bad = 0, v[7], st = 0;
    void *in = getp(a[0], &bad), *w = getp(a[1], &bad);
    for (int i = 0; i < 7; ++i) v[i] = geti(a[2 + i], &bad);
    void *b = getp(a[9], &bad);
    const int relu = geti(a[10], &bad);
    void *y = getp(a[11], &bad), *s = getp(a[12], &bad);
    CALL(L.conv_si(in, w, v[0], v[1], v[2], v[3], v[4], v[5], v[6], b, relu, y, s));
    return PyLong_FromLong(st);
}

/* conv_sip(in, dense, sh, sw, ph, pw, bias, relu, y, variant, stream) -> status */
static PyObject *py_conv_sip(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    if (wrong_count(n, 11)) return NULL;
    int bad = 0, v[4], st = 0;
    void *in = getp(a[0], &bad), *d = getp(a[1], &bad);
    for (int i = 0; i < 4; ++i) v[i] = geti(a[2 + i], &bad);
    void *b = getp(a[6], &bad);
    const int relu = geti(a[7], &bad);
    void *y = getp(a[8], &bad);
    const int var = geti(a[9], &bad);
    void *s = getp(a[10], &bad);
    CALL(L.conv_sip(in, d, v[0], v[1], v[2], v[3], b, relu, y, var, s));
    return PyLong_FromLong(st);
}

/* compress(kind, src, d0, d1, d2, d3, stream) -> (status, handle, nnz); kind 0: filters K, C, R, S; 1: activation N, C, H, W */
static PyObject *py_compress(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    if (wrong_count(n, 7)) return NULL;
    int bad = 0, v[4], st = 0;
    const int kind = geti(a[0], &bad);
    void *src = getp(a[1], &bad);
    for (int i = 0; i < 4; ++i) v[i] = geti(a[2 + i], &bad);
    void *s = getp(a[6], &bad);
    void *h = NULL;
    long long nnz = 0;
    CALL(kind == 0 ? L.filter_compress(src, v[0], v[1], v[2], v[3], s, (fscnn_filter_t **)&h)
                   : L.input_compress(src, v[0], v[1], v[2], v[3], s, (fscnn_input_t **)&h));
    if (st == 0) {
        if (kind == 0) L.filter_info(h, NULL, NULL, NULL, NULL, &nnz);
        else L.input_info(h, NULL, NULL, NULL, NULL, &nnz);
    }
    return Py_BuildValue("iNL", st, PyLong_FromVoidPtr(h), nnz);
}

/* transpose(rowptr, idx, val, dims, nnz, tptr, tidx, tval, ws, ws_bytes, stream) -> status; two dims: matrix, three: tensor */
static PyObject *py_transpose(PyObject *self, PyObject *const *a, Py_ssize_t n)
{
    if (wrong_count(n, 11)) return NULL;
    int bad = 0, d[3] = {0, 0, 0}, st = 0;
    void *p[3] = {getp(a[0], &bad), getp(a[1], &bad), getp(a[2], &bad)};
    if (!PyTuple_Check(a[3]) || PyTuple_GET_SIZE(a[3]) < 2 || PyTuple_GET_SIZE(a[3]) > 3) {
        PyErr_SetString(PyExc_TypeError, "dims: a tuple of two or three ints");
        return NULL;
    }
    const int nd = (int)PyTuple_GET_SIZE(a[3]);
    for (int i = 0; i < nd; ++i) d[i] = geti(PyTuple_GET_ITEM(a[3], i), &bad);
    const long long nnz = PyLong_AsLongLong(a[4]);
    void *t[4] = {getp(a[5], &bad), getp(a[6], &bad), getp(a[7], &bad), getp(a[8], &bad)};
    const long long bytes = PyLong_AsLongLong(a[9]);
    void *s = getp(a[10], &bad);
    if (PyErr_Occurred()) bad = 1;
    CALL(nd == 2 ? L.transpose(p[0], p[1], p[2], d[0], d[1], nnz, t[0], t[1], t[2], t[3], bytes, s)
                 : L.tensor_transpose(p[0], p[1], p[2], d[0], d[1], d[2], nnz, t[0], t[1], t[2], t[3], bytes, s));
    return PyLong_FromLong(st);
}

#define FAST(name, fn) {name, (PyCFunction)(void (*)(void))fn, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {
    {"bind", py_bind, METH_O, NULL},
    FAST("conv", py_conv), FAST("emit", py_emit), FAST("conv_si", py_conv_si), FAST("conv_sip", py_conv_sip),
    FAST("compress", py_compress), FAST("transpose", py_transpose),
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fscnn_call", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__fscnn_call(void) { return PyModule_Create(&module); }
