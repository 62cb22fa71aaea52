/*
 * smol_pycall.c -- the Python binding's call into libsmol, as a CPython
 * extension module (_smolcall).
 *
 * call(address, *args) calls the C function at `address` with up to 18
 * integer or pointer arguments and returns its int result: None is a null
 * pointer or zero, an int itself, any other object the address of its
 * C-contiguous buffer (numpy arrays, ctypes structures), held for the call. The
 * GIL is released meanwhile. An ABI function takes only such arguments, which
 * the x86-64 System V convention passes in 64-bit registers and stack slots.
 *
 * Taking a numpy array's address through its `ctypes` attribute costs 0.7 us
 * and ctypes' own conversion of ten arguments 0.6; here a call of three tables
 * costs 0.4 us in all.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#define MAX_ARGS 18

typedef int64_t w;
typedef int (*Fn)(w, w, w, w, w, w, w, w, w, w, w, w, w, w, w, w, w, w);

static PyObject *call(PyObject *self, PyObject *const *args, Py_ssize_t nargs)
{
    (void)self;
    if (nargs < 1 || nargs > MAX_ARGS + 1) {
        PyErr_Format(PyExc_TypeError, "call(address, ...) takes up to %d arguments", MAX_ARGS);
        return NULL;
    }
    const Fn fn = (Fn)PyLong_AsVoidPtr(args[0]);
    if (!fn) {
        if (!PyErr_Occurred())
            PyErr_SetString(PyExc_ValueError, "null function address");
        return NULL;
    }
    w a[MAX_ARGS] = {0};
    Py_buffer views[MAX_ARGS];
    int nviews = 0, result = 0, ok = 1;
    for (Py_ssize_t i = 1; i < nargs && ok; ++i) {
        PyObject *o = args[i];
        if (o == Py_None)
            continue;
        if (PyLong_Check(o)) {
            int overflow = 0;
            a[i - 1] = PyLong_AsLongLongAndOverflow(o, &overflow);
            if (overflow > 0) /* addresses above 2^63 */
                a[i - 1] = (w)PyLong_AsUnsignedLongLong(o);
            ok = overflow >= 0 && !PyErr_Occurred();
            if (overflow < 0)
                PyErr_SetString(PyExc_OverflowError, "integer argument below -2^63");
        } else if (PyObject_GetBuffer(o, &views[nviews], PyBUF_ND) == 0) {
            const Py_buffer *v = &views[nviews++];
            a[i - 1] = (w)(intptr_t)v->buf;
            if (v->ndim == 0 && PyIndex_Check(o)) {
                /* a numpy integer: a number whose address nobody means */
                PyErr_Format(PyExc_TypeError, "argument %zd is a %.80s, not an int", i,
                             Py_TYPE(o)->tp_name);
                ok = 0;
            }
        } else {
            ok = 0;
        }
    }
    if (ok) {
        /* Arguments past the callee's own are not read by it. */
        Py_BEGIN_ALLOW_THREADS
        result = fn(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11],
                    a[12], a[13], a[14], a[15], a[16], a[17]);
        Py_END_ALLOW_THREADS
    }
    while (nviews > 0)
        PyBuffer_Release(&views[--nviews]);
    return ok ? PyLong_FromLong(result) : NULL;
}

static PyMethodDef methods[] = {
    {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL,
     "call(address, *args) -> int: call a C function with integer and buffer arguments."},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_smolcall", NULL, -1, methods,
                                    NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__smolcall(void) { return PyModule_Create(&module); }
