/* The check of one tensor argument, for binding.py, six or so of which a call makes: 0.6 us each in Python, 0.22 here.  A
 * client-server cycle (19 calls, 25 launches), which the host bounds: 151 -> 146 us enqueued and in all, of which the GPU needs
 * 96 when it never waits.  The stable CPython API; whatever the tensor's
 * attributes say, they say here as they would there. */
#define PY_SSIZE_T_CLEAN
#define Py_LIMITED_API 0x030a0000      /* CPython 3.10 and later load the same file */
#include <Python.h>

static PyObject *tensor_type, *s_is_cuda, *s_is_contiguous, *s_dtype, *s_numel, *s_data_ptr;
static PyObject *is_contiguous, *numel, *data_ptr;     /* torch.Tensor's own, for what is no subclass of it */

static PyObject *call(PyObject *t, int plain, PyObject *method, PyObject *name)
{
    return plain ? PyObject_CallFunctionObjArgs(method, t, NULL) : PyObject_CallMethodObjArgs(t, name, NULL);
}

/* 1, 0, or -1 with an exception */
static int truth(PyObject *o)
{
    if (!o) return -1;
    const int r = PyObject_IsTrue(o);
    Py_DECREF(o);
    return r;
}

/* dev(tensor or None, dtype, numel, name) -> address or None: a contiguous CUDA tensor of that type with at least that many elements */
static PyObject *dev(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    (void)self;
    if (n != 4) return PyErr_Format(PyExc_TypeError, "dev: 4 arguments expected, not %zd", n);
    PyObject *t = args[0], *name = args[3];
    if (t == Py_None) Py_RETURN_NONE;
    const int plain = (PyObject *)Py_TYPE(t) == tensor_type;
    if (!plain) {
        const int is = PyObject_IsInstance(t, tensor_type);
        if (is < 0) return NULL;
        if (!is) return PyErr_Format(PyExc_TypeError, "%S: expected a torch tensor", name);
    }
    int ok = truth(PyObject_GetAttr(t, s_is_cuda));
    if (ok > 0) ok = truth(call(t, plain, is_contiguous, s_is_contiguous));
    if (ok < 0) return NULL;
    if (!ok) return PyErr_Format(PyExc_ValueError, "%S: must be a contiguous CUDA tensor", name);
    PyObject *dtype = PyObject_GetAttr(t, s_dtype);
    if (!dtype) return NULL;
    if (dtype != args[1]) {
        const int differ = PyObject_RichCompareBool(dtype, args[1], Py_NE);
        if (differ > 0) PyErr_Format(PyExc_ValueError, "%S: dtype %S, expected %S", name, dtype, args[1]);
        if (differ) {
            Py_DECREF(dtype);
            return NULL;
        }
    }
    Py_DECREF(dtype);
    PyObject *have = call(t, plain, numel, s_numel);
    if (!have) return NULL;
    const int less = PyObject_RichCompareBool(have, args[2], Py_LT);
    if (less > 0) PyErr_Format(PyExc_ValueError, "%S: %S elements, the call touches %S", name, have, args[2]);
    Py_DECREF(have);
    if (less) return NULL;
    return call(t, plain, data_ptr, s_data_ptr);
}

static PyMethodDef methods[] = {
    {"dev", (PyCFunction)(void (*)(void))dev, METH_FASTCALL,
     "Device pointer (a number: the argument types make the pointer) of a tensor after checking it can hold what the call touches."},
    {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_argcheck", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__argcheck(void)
{
    PyObject *torch = PyImport_ImportModule("torch");
    if (!torch) return NULL;
    tensor_type = PyObject_GetAttrString(torch, "Tensor");
    Py_DECREF(torch);
    if (!tensor_type) return NULL;
    is_contiguous = PyObject_GetAttrString(tensor_type, "is_contiguous");
    numel = PyObject_GetAttrString(tensor_type, "numel");
    data_ptr = PyObject_GetAttrString(tensor_type, "data_ptr");
    if (!is_contiguous || !numel || !data_ptr) return NULL;
    s_is_cuda = PyUnicode_InternFromString("is_cuda");
    s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    s_dtype = PyUnicode_InternFromString("dtype");
    s_numel = PyUnicode_InternFromString("numel");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    if (!s_is_cuda || !s_is_contiguous || !s_dtype || !s_numel || !s_data_ptr) return NULL;
    return PyModule_Create(&module);
}
