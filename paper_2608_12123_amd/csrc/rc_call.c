/* rc_call.c -- CPython side of the calls that run once per launch.
 *
 * A launch of a small cohort costs the GPU under 4 us and HIP about 3.5 us of
 * host time; marshalled by ctypes (eight converted arguments) and with a
 * stream object made for each call, it cost the host 7.1 us.  call() passes
 * the same arguments to the same C entry point in about 0.3 us:
 *
 *   bind(handle_type, buffers_type)
 *   call(fn, handle, buffers, a0, a1, a2, a3, a4, stream) -> status
 *
 * fn is the address of the entry point; handle a handle_type (ctypes'
 * c_void_p), an address or None; buffers a buffers_type (the ctypes structure
 * of an rc_buffers); a0..a4 integers, taken modulo 2^32 as ctypes takes a
 * c_uint32; stream an address or None.  Any other form is a TypeError, and
 * the binding hands it to ctypes, which converts or refuses it by its own
 * rules.  The interpreter lock is released during the call.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <string.h>

#include "rc_cohort.h"

typedef int (*chain_fn)(rc_cohort *, const rc_buffers *, uint32_t, uint32_t, int, uint32_t, uint32_t, void *);

static PyTypeObject *handle_type, *buffers_type;

static PyObject *bind(PyObject *self, PyObject *args)
{
    PyTypeObject *h, *b;
    (void)self;
    if (!PyArg_ParseTuple(args, "O!O!", &PyType_Type, &h, &PyType_Type, &b)) return NULL;
    Py_INCREF(h);
    Py_INCREF(b);
    Py_XDECREF(handle_type);
    Py_XDECREF(buffers_type);
    handle_type = h;
    buffers_type = b;
    Py_RETURN_NONE;
}

/* An address from None, an integer (modulo the address size, as ctypes takes
 * one) or a handle_type. */
static int as_pointer(PyObject *o, void **out)
{
    if (o == Py_None) {
        *out = NULL;
        return 0;
    }
    if (PyLong_Check(o)) {
        *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
        return PyErr_Occurred() ? -1 : 0;
    }
    if (!handle_type || !PyObject_TypeCheck(o, handle_type)) {
        PyErr_SetString(PyExc_TypeError, "not a pointer");
        return -1;
    }
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) return -1;
    const int ok = b.len == (Py_ssize_t)sizeof(void *);
    if (ok) memcpy(out, b.buf, sizeof(void *));
    PyBuffer_Release(&b);
    if (!ok) PyErr_SetString(PyExc_TypeError, "not a pointer");
    return ok ? 0 : -1;
}

static PyObject *call(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    (void)self;
    if (n != 9) {
        PyErr_SetString(PyExc_TypeError, "call() takes 9 arguments");
        return NULL;
    }
    void *fn, *handle, *stream;
    uint32_t v[5];
    if (as_pointer(args[0], &fn) != 0 || as_pointer(args[1], &handle) != 0 || as_pointer(args[8], &stream) != 0)
        return NULL;
    for (int i = 0; i < 5; ++i) {
        v[i] = (uint32_t)PyLong_AsUnsignedLongMask(args[3 + i]);
        if (PyErr_Occurred()) return NULL;
    }
    if (!fn) {
        PyErr_SetString(PyExc_ValueError, "no entry point");
        return NULL;
    }
    Py_buffer b; /* held during the call */
    if (!buffers_type || !PyObject_TypeCheck(args[2], buffers_type)) {
        PyErr_SetString(PyExc_TypeError, "buffers is not an RcBuffers");
        return NULL;
    }
    if (PyObject_GetBuffer(args[2], &b, PyBUF_SIMPLE) != 0) return NULL;
    if (b.len < (Py_ssize_t)sizeof(rc_buffers)) { /* a subclass may hold more */
        PyBuffer_Release(&b);
        PyErr_SetString(PyExc_TypeError, "buffers is not an RcBuffers");
        return NULL;
    }
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = ((chain_fn)(uintptr_t)fn)((rc_cohort *)handle, (const rc_buffers *)b.buf, v[0], v[1], (int)v[2], v[3], v[4],
                                       stream);
    Py_END_ALLOW_THREADS
    PyBuffer_Release(&b);
    return PyLong_FromLong(status);
}

static PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, "bind(handle_type, buffers_type): the types that call() takes"},
    {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL,
     "call(fn, handle, buffers, a0, a1, a2, a3, a4, stream): the status of a chain entry point"},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rc_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__rc_call(void) { return PyModule_Create(&module); }
