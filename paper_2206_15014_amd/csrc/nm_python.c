/* Argument marshalling of the hot calls of binding.py in C: tensor -> pointer, shape and row stride by the tensor's own
 * methods, the current stream's handle, then the call itself with the interpreter lock released.  A forward pass of a
 * compressed encoder on one short sentence is 96 calls of a few microseconds each, so what the interpreter and ctypes spend per call
 * is what such a pass takes: 4.5 us of a call's 6.0 were marshalling, here 1.4; one 768 x 768 layer on 128 tokens 6.0 -> 4.5 us,
 * BERT-large on 128 tokens 563 -> 457 us a pass, which is what its launches take.
 *
 * A function returns the library's status, or None where an argument is not what it takes (a float for a dimension, say): the
 * caller then goes through ctypes, which decides as it always has.  Exceptions of the tensors' methods pass through.
 * No torch header is needed and the module does not link against libnm: bind() hands it the entry points' addresses. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "nm.h"

static int (*gemm_fn)(const int8_t*, int, int, int, float, const float*, const void*, const void*, const float*, int, int, int, int, int,
                      const float*, int32_t*, void*, int, int, void*);
static PyObject *s_data_ptr, *s_stride, *s_shape, *zero;

enum { BAD = -1, NO = 0, YES = 1 };            /* an exception is set; not for us; converted */

/* None, an address or a tensor -> pointer */
static int to_ptr(PyObject* o, void** out)
{
    if (o == Py_None) {
        *out = NULL;
        return YES;
    }
    if (PyLong_Check(o)) {
        *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
        return YES;
    }
    PyObject* p = PyObject_CallMethodNoArgs(o, s_data_ptr);
    if (!p) return BAD;
    const int ok = PyLong_Check(p);
    if (ok) *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    return ok ? YES : NO;
}

static int to_int(PyObject* o, int* out)
{
    if (!PyLong_Check(o)) return NO;
    *out = (int)PyLong_AsUnsignedLongMask(o);  /* ctypes' conversion: the low bits */
    return YES;
}

static int to_float(PyObject* o, float* out)
{
    if (!PyFloat_Check(o) && !PyLong_Check(o)) return NO;
    const double d = PyFloat_AsDouble(o);
    if (d == -1.0 && PyErr_Occurred()) return BAD;
    *out = (float)d;
    return YES;
}

static int row_stride(PyObject* t, int* out)
{
    PyObject* s = PyObject_CallMethodOneArg(t, s_stride, zero);
    if (!s) return BAD;
    const int ok = to_int(s, out);
    Py_DECREF(s);
    return ok;
}

static int shape_2d(PyObject* t, int* rows, int* cols)
{
    PyObject* s = PyObject_GetAttr(t, s_shape);
    if (!s) return BAD;
    int ok = NO;
    if (PyTuple_Check(s) && PyTuple_GET_SIZE(s) == 2) ok = to_int(PyTuple_GET_ITEM(s, 0), rows) && to_int(PyTuple_GET_ITEM(s, 1), cols) ? YES : NO;
    Py_DECREF(s);
    return ok;
}

#define TRY(conversion) \
    do { \
        const int r_ = (conversion); \
        if (r_ == BAD) return NULL; \
        if (r_ == NO) Py_RETURN_NONE; \
    } while (0)

/* gemm(X, act_scale, vals, meta, scales, O, N, M, bits, bias, acc, out, out_dtype, ldo, stream, layout, act_scale_dev): nm_gemm's
 * arguments, the stream as its handle */
static PyObject* py_gemm(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    int tokens, K, ldx, O, N, M, bits, out_dtype, ldo, layout;
    float act_scale;
    void *X, *vals, *meta, *scales, *bias, *acc, *out, *stream, *act_scale_dev;
    if (n != 17 || !gemm_fn) Py_RETURN_NONE;
    TRY(to_int(a[5], &O));
    TRY(to_int(a[6], &N));
    TRY(to_int(a[7], &M));
    TRY(to_int(a[8], &bits));
    TRY(to_int(a[12], &out_dtype));
    TRY(to_int(a[15], &layout));
    TRY(to_float(a[1], &act_scale));
    TRY(shape_2d(a[0], &tokens, &K));
    if (a[13] == Py_None) {
        PyObject* ref = a[11] != Py_None ? a[11] : a[10];
        if (ref == Py_None || !PyObject_HasAttr(ref, s_stride)) ldo = O;
        else TRY(row_stride(ref, &ldo));
    } else {
        TRY(to_int(a[13], &ldo));
    }
    TRY(to_ptr(a[0], &X));
    TRY(row_stride(a[0], &ldx));
    TRY(to_ptr(a[16], &act_scale_dev));
    TRY(to_ptr(a[2], &vals));
    TRY(to_ptr(a[3], &meta));
    TRY(to_ptr(a[4], &scales));
    TRY(to_ptr(a[9], &bias));
    TRY(to_ptr(a[10], &acc));
    TRY(to_ptr(a[11], &out));
    if (!PyLong_Check(a[14])) Py_RETURN_NONE;
    stream = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(a[14]);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = gemm_fn(X, tokens, K, ldx, act_scale, act_scale_dev, vals, meta, scales, O, N, M, bits, layout, bias, acc, out, out_dtype, ldo, stream);
    Py_END_ALLOW_THREADS
    (void)self;
    return PyLong_FromLong(rc);
}

/* bind(address of nm_gemm) */
static PyObject* py_bind(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    (void)self;
    if (n != 1 || !PyLong_Check(a[0])) {
        PyErr_SetString(PyExc_TypeError, "bind(address of nm_gemm)");
        return NULL;
    }
    *(void**)&gemm_fn = (void*)(uintptr_t)PyLong_AsUnsignedLongLongMask(a[0]);
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {{"bind", (PyCFunction)(void (*)(void))py_bind, METH_FASTCALL, NULL},
                                {"gemm", (PyCFunction)(void (*)(void))py_gemm, METH_FASTCALL, NULL},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nm_python", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__nm_python(void)
{
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_stride = PyUnicode_InternFromString("stride");
    s_shape = PyUnicode_InternFromString("shape");
    zero = PyLong_FromLong(0);
    if (!s_data_ptr || !s_stride || !s_shape || !zero) return NULL;
    return PyModule_Create(&module);
}
