// CPython extension: calls of the library's C functions with the arguments a decode step has in hand (torch tensors, numpy
// arrays, ctypes structures, integers), without an object per argument.  The smallest steps are bound by the host, where ctypes took
// 2.3 us to convert the seventeen arguments of an attention call; binding.py has the figures of whole calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#if !defined(__x86_64__) || defined(_WIN32)
#error "call() passes every argument as 64 bits, which the System V calling convention of x86-64 allows (build.py leaves the file out elsewhere)"
#endif

static PyObject *g_ndarray, *g_structure, *g_data_ptr;

// call(function address, kinds, other, arguments...) -> int.  kinds, a byte per argument: a an address given as an integer, None (NULL), an
// array or a tensor; p one given as an integer or None; s a ctypes structure; i an integer.  An argument of any other type: other is
// called with all of them and its result returned, so that what is taken and what is refused is for it to say.
enum { kMost = 17 };

// 1: converted, 0: not a type of this kind, -1: an exception is set
static int integer(PyObject* x, uint64_t* out) {
    if (!PyLong_Check(x)) return 0;
    *out = PyLong_AsUnsignedLongLongMask(x);
    return *out == (uint64_t)-1 && PyErr_Occurred() ? -1 : 1;
}

static int buffer(PyObject* x, uint64_t* out) {
    Py_buffer view;
    if (PyObject_GetBuffer(x, &view, PyBUF_STRIDED_RO)) {    // (arrays of dates, for instance, have an address but no buffer)
        PyErr_Clear();
        return 0;
    }
    *out = (uint64_t)(uintptr_t)view.buf;                // the caller holds the object during the call
    PyBuffer_Release(&view);
    return 1;
}

static int convert(char kind, PyObject* x, uint64_t* out) {
    if (kind == 's') return PyObject_TypeCheck(x, (PyTypeObject*)g_structure) ? buffer(x, out) : 0;
    if (kind != 'i' && x == Py_None) {
        *out = 0;
        return 1;
    }
    const int rc = integer(x, out);
    if (rc || kind != 'a') return rc;
    if (PyObject_TypeCheck(x, (PyTypeObject*)g_ndarray)) return buffer(x, out);
    PyObject* at = PyObject_CallMethodNoArgs(x, g_data_ptr);
    if (!at) {
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
        PyErr_Clear();
        return 0;
    }
    const int done = integer(at, out);
    Py_DECREF(at);
    return done;
}

typedef uint64_t U;
static PyObject* call(PyObject* self, PyObject* const* args, Py_ssize_t n_args) {
    (void)self;
    U a[kMost] = {0};
    char* kinds;
    Py_ssize_t n;
    if (n_args < 3 || PyBytes_AsStringAndSize(args[1], &kinds, &n)) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "a function address, argument kinds and a function are required");
        return NULL;
    }
    if (n != n_args - 3 || n > kMost) {
        PyErr_Format(PyExc_TypeError, "%zd arguments are required, not %zd", n, n_args - 3);
        return NULL;
    }
    U f;
    const int known = integer(args[0], &f);
    if (known <= 0) {
        if (known == 0) PyErr_SetString(PyExc_TypeError, "the function address is not an integer");
        return NULL;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        const int done = convert(kinds[i], args[3 + i], &a[i]);
        if (done < 0) return NULL;
        if (done == 0) return PyObject_Vectorcall(args[2], args + 3, (size_t)n, NULL);
    }
    int rc;
    // Every argument is an integer or an address and so has a register or eight bytes of stack of its own.
    Py_BEGIN_ALLOW_THREADS
    if (n <= 3) rc = ((int (*)(U, U, U))f)(a[0], a[1], a[2]);
    else if (n <= 7) rc = ((int (*)(U, U, U, U, U, U, U))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6]);
    else if (n <= 12) rc = ((int (*)(U, U, U, U, U, U, U, U, U, U, U, U))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11]);
    else
        rc = ((int (*)(U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U, U))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11],
                                                                            a[12], a[13], a[14], a[15], a[16]);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// init(array type, type of ctypes structures)
static PyObject* init(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    (void)self;
    if (n != 2 || !PyType_Check(args[0]) || !PyType_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "two types are required");
        return NULL;
    }
    Py_INCREF(args[0]);
    Py_INCREF(args[1]);
    Py_XDECREF(g_ndarray);
    Py_XDECREF(g_structure);
    g_ndarray = args[0];
    g_structure = args[1];
    Py_RETURN_NONE;
}

static PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, NULL},
                                {"init", (PyCFunction)(void (*)(void))init, METH_FASTCALL, NULL},
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_apt_call", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__apt_call(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    return g_data_ptr ? PyModule_Create(&module) : NULL;
}
