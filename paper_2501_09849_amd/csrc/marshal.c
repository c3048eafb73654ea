/*
 * The calls of libcdl as functions of a Python module: arguments from tensors and numbers to pointers and C values, the
 * library's function, its status back.  A training step of a small layer is half a dozen calls of a few microseconds of
 * GPU time each, so what Python spends per call counts: 7 us with ctypes (two Python-level calls per tensor, a Stream
 * object, a struct, ctypes' own conversion of fifteen arguments), 1.5 us here.
 *
 * Tensors are used through their methods only (is_contiguous, data_ptr, nbytes); addresses of the library's functions
 * come from the caller (init), which has loaded the library.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "cdl.h"

static PyObject *s_data_ptr, *s_is_contiguous, *s_nbytes, *s_cuda_stream;
static PyObject *f_raw_stream, *f_device;      /* current stream of a device, current device */

/* address of a tensor; None = NULL, an integer is an address */
static int get_ptr(PyObject *o, void **p)
{
    if (o == Py_None) { *p = NULL; return 0; }
    if (PyLong_Check(o)) { *p = PyLong_AsVoidPtr(o); return PyErr_Occurred() ? -1 : 0; }
    PyObject *c = PyObject_CallMethodNoArgs(o, s_is_contiguous);
    if (!c) return -1;
    const int yes = PyObject_IsTrue(c);
    Py_DECREF(c);
    if (yes < 0) return -1;
    if (!yes) { PyErr_SetString(PyExc_ValueError, "tensor must be contiguous"); return -1; }
    PyObject *a = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!a) return -1;
    *p = PyLong_AsVoidPtr(a);
    Py_DECREF(a);
    return PyErr_Occurred() ? -1 : 0;
}

static int get_ws(PyObject *o, void **p, size_t *bytes)
{
    if (o == Py_None) { *p = NULL; *bytes = 0; return 0; }
    PyObject *a = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!a) return -1;
    *p = PyLong_AsVoidPtr(a);
    Py_DECREF(a);
    PyObject *n = PyObject_GetAttr(o, s_nbytes);
    if (!n) return -1;
    *bytes = PyLong_AsSize_t(n);
    Py_DECREF(n);
    return PyErr_Occurred() ? -1 : 0;
}

static int get_stream(PyObject *o, void **p)
{
    if (o == Py_None) {
        PyObject *d = PyObject_CallNoArgs(f_device);
        if (!d) return -1;
        PyObject *s = PyObject_CallOneArg(f_raw_stream, d);
        Py_DECREF(d);
        if (!s) return -1;
        *p = PyLong_AsVoidPtr(s);
        Py_DECREF(s);
    } else if (PyLong_Check(o)) {
        *p = PyLong_AsVoidPtr(o);
    } else {
        PyObject *s = PyObject_GetAttr(o, s_cuda_stream);
        if (!s) return -1;
        *p = PyLong_AsVoidPtr(s);
        Py_DECREF(s);
    }
    return PyErr_Occurred() ? -1 : 0;
}

/*
 * An integer.  Sizes are integers or what Python takes as an index (a float or a text would be a wrong length without a word);
 * the numbers of a quantizer and offsets are converted as int() does.
 */
static int get_int_by(PyObject *o, int64_t *v, PyObject *(*convert)(PyObject *))
{
    if (PyLong_Check(o)) { *v = (int64_t)PyLong_AsUnsignedLongLongMask(o); return PyErr_Occurred() ? -1 : 0; }
    PyObject *n = convert(o);
    if (!n) return -1;
    *v = (int64_t)PyLong_AsUnsignedLongLongMask(n);
    Py_DECREF(n);
    return PyErr_Occurred() ? -1 : 0;
}
static int get_index(PyObject *o, int64_t *v) { return get_int_by(o, v, PyNumber_Index); }
static int get_int(PyObject *o, int64_t *v) { return get_int_by(o, v, PyNumber_Long); }

/* a real number of a quantizer, or a scale: as float() converts it */
static int get_real(PyObject *o, float *v)
{
    if (PyFloat_Check(o)) { *v = (float)PyFloat_AS_DOUBLE(o); return 0; }
    PyObject *f = PyNumber_Float(o);
    if (!f) return -1;
    *v = (float)PyFloat_AsDouble(f);
    Py_DECREF(f);
    return PyErr_Occurred() ? -1 : 0;
}

/*
 * One call's arguments by the letters of a format: p pointer, n 64-bit size, i 32-bit size, o offset (among the 32-bit
 * integers), f float, r real number by float() (among the floats), q quantizer (lo, n_levels, delta, alpha, top_k: five
 * arguments), w workspace (pointer and size), s stream.  They are filled in order into the arrays of their kind.
 */
struct args {
    void *p[12];
    int64_t n;
    int32_t i[12];
    float f[2];
    cdl_qparams q[2];
    void *ws;
    size_t ws_bytes;
    void *stream;
};

static int parse(const char *name, const char *format, PyObject *const *o, Py_ssize_t count, struct args *a)
{
    int np = 0, ni = 0, nf = 0, nq = 0;
    Py_ssize_t at = 0;
    int64_t v;
    for (const char *c = format; *c; ++c) {
        if (at + (*c == 'q' ? 5 : 1) > count) goto wrong;
        switch (*c) {
            case 'p': if (get_ptr(o[at++], &a->p[np++])) return -1; break;
            case 'n': if (get_index(o[at++], &a->n)) return -1; break;
            case 'i': if (get_index(o[at++], &v)) return -1; a->i[ni++] = (int32_t)v; break;
            case 'o': if (get_int(o[at++], &v)) return -1; a->i[ni++] = (int32_t)v; break;
            case 'r': if (get_real(o[at++], &a->f[nf++])) return -1; break;
            case 'f': a->f[nf] = (float)PyFloat_AsDouble(o[at++]); ++nf; if (PyErr_Occurred()) return -1; break;
            case 'q': {
                cdl_qparams *q = &a->q[nq++];
                if (get_int(o[at], &v)) return -1;
                q->lo = (int32_t)v;
                if (get_int(o[at + 1], &v)) return -1;
                q->n_levels = (int32_t)v;
                if (get_real(o[at + 2], &q->delta) || get_real(o[at + 3], &q->alpha) || get_int(o[at + 4], &v)) return -1;
                q->top_k = (int32_t)v;
                at += 5;
                break;
            }
            case 'w': if (get_ws(o[at++], &a->ws, &a->ws_bytes)) return -1; break;
            case 's': if (get_stream(o[at++], &a->stream)) return -1; break;
        }
    }
    if (at == count) return 0;
wrong:
    PyErr_Format(PyExc_TypeError, "%s: wrong number of arguments (%zd)", name, count);
    return -1;
}

/* the library's functions, and for each a Python function NAME(arguments by FORMAT) -> status */
#define CALLS(X)                                                                                                                        \
    X(cdl_quantize_fwd, "pnqppppws", (a.p[0], a.n, &a.q[0], a.p[1], a.p[2], a.p[3], a.p[4], a.ws, a.ws_bytes, a.stream))                \
    X(cdl_quantize_bwd, "ppnqpppws", (a.p[0], a.p[1], a.n, &a.q[0], a.p[2], a.p[3], a.p[4], a.ws, a.ws_bytes, a.stream))                \
    X(cdl_marginal_entropy, "pnqppws", (a.p[0], a.n, &a.q[0], a.p[1], a.p[2], a.ws, a.ws_bytes, a.stream))                              \
    X(cdl_quantize_draw, "ppnqps", (a.p[0], a.p[1], a.n, &a.q[0], a.p[2], a.stream))                                                    \
    X(cdl_entropy_bwd, "pppnqrpppws", (a.p[0], a.p[1], a.p[2], a.n, &a.q[0], a.f[0], a.p[3], a.p[4], a.p[5], a.ws, a.ws_bytes, a.stream)) \
    X(cdl_huffman_bits, "pniipppws", (a.p[0], a.n, a.i[0], a.i[1], a.p[1], a.p[2], a.p[3], a.ws, a.ws_bytes, a.stream))                 \
    X(cdl_qgemm_fwd_offset, "ppiiiffooppws",                                                                                            \
      (a.p[0], a.p[1], a.i[0], a.i[1], a.i[2], a.f[0], a.f[1], a.i[3], a.i[4], a.p[2], a.p[3], a.ws, a.ws_bytes, a.stream))             \
    X(cdl_qgemm_bwd_offset, "pppiiiffooppws",                                                                                           \
      (a.p[0], a.p[1], a.p[2], a.i[0], a.i[1], a.i[2], a.f[0], a.f[1], a.i[3], a.i[4], a.p[3], a.p[4], a.ws, a.ws_bytes, a.stream))     \
    X(cdl_qgemm_fwd_quantize, "pqpiiifps", (a.p[0], &a.q[0], a.p[1], a.i[0], a.i[1], a.i[2], a.f[0], a.p[2], a.stream))                 \
    X(cdl_qconv_fwd, "ppiiiiiiiiiffoppws",                                                                                              \
      (a.p[0], a.p[1], a.i[0], a.i[1], a.i[2], a.i[3], a.i[4], a.i[5], a.i[6], a.i[7], a.i[8], a.f[0], a.f[1], a.i[9], a.p[2], a.p[3],  \
       a.ws, a.ws_bytes, a.stream))                                                                                                     \
    X(cdl_qconv_bwd_weights, "ppiiiiiiiiifopws",                                                                                        \
      (a.p[0], a.p[1], a.i[0], a.i[1], a.i[2], a.i[3], a.i[4], a.i[5], a.i[6], a.i[7], a.i[8], a.f[0], a.i[9], a.p[2], a.ws,            \
       a.ws_bytes, a.stream))                                                                                                           \
    X(cdl_qconv_bwd_activations, "ppiiiiiiiiifpws",                                                                                     \
      (a.p[0], a.p[1], a.i[0], a.i[1], a.i[2], a.i[3], a.i[4], a.i[5], a.i[6], a.i[7], a.i[8], a.f[0], a.p[2], a.ws, a.ws_bytes,        \
       a.stream))                                                                                                                       \
    /* the last integer: whether the weight quantizer is given */                                                                       \
    X(cdl_qgemm_bwd_quantize_bwd, "pppiiipqfopppppiqpppws",                                                                             \
      (a.p[0], a.p[1], a.p[2], a.i[0], a.i[1], a.i[2], a.p[3], &a.q[0], a.f[0], a.i[3], a.p[4], a.p[5], a.p[6], a.p[7], a.p[8],         \
       a.i[4] ? &a.q[1] : NULL, a.p[9], a.p[10], a.p[11], a.ws, a.ws_bytes, a.stream))

#define DEFINE(NAME, FORMAT, ARGS)                                                                  \
    static __typeof__(&NAME) fn_##NAME;                                                             \
    static PyObject *py_##NAME(PyObject *self, PyObject *const *o, Py_ssize_t count)                \
    {                                                                                               \
        struct args a;                                                                              \
        int rc;                                                                                     \
        (void)self;                                                                                 \
        if (!fn_##NAME) { PyErr_SetString(PyExc_RuntimeError, "libcdl is not loaded"); return NULL; } \
        if (parse(#NAME, FORMAT, o, count, &a)) return NULL;                                        \
        Py_BEGIN_ALLOW_THREADS                                                                      \
        rc = fn_##NAME ARGS;                                                                        \
        Py_END_ALLOW_THREADS                                                                        \
        return PyLong_FromLong(rc);                                                                 \
    }
CALLS(DEFINE)

/* init({name: address}, function of a device's current stream, function of the current device) */
static PyObject *init(PyObject *self, PyObject *args)
{
    PyObject *table, *raw, *dev;
    (void)self;
    if (!PyArg_ParseTuple(args, "O!OO", &PyDict_Type, &table, &raw, &dev)) return NULL;
#define TAKE(NAME, FORMAT, ARGS)                                                                    \
    {                                                                                               \
        PyObject *v = PyDict_GetItemString(table, #NAME);                                           \
        void *p = v ? PyLong_AsVoidPtr(v) : NULL;                                                   \
        if (!p) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #NAME); return NULL; }     \
        fn_##NAME = (__typeof__(fn_##NAME))p;                                                       \
    }
    CALLS(TAKE)
    Py_INCREF(raw);
    Py_INCREF(dev);
    Py_XDECREF(f_raw_stream);
    Py_XDECREF(f_device);
    f_raw_stream = raw;
    f_device = dev;
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
#define METHOD(NAME, FORMAT, ARGS) {#NAME, (PyCFunction)(void (*)(void))py_##NAME, METH_FASTCALL, FORMAT},
    CALLS(METHOD){"init", init, METH_VARARGS, "function addresses of libcdl by name, and torch's stream and device queries"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "libcdl calls", -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__marshal(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_nbytes = PyUnicode_InternFromString("nbytes");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return PyModule_Create(&module);
}
