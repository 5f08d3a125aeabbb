/*
 * Native marshalling of the four calls a training loop makes every step (rb_update, rb_sample_augment, rb_update_sample,
 * rb_announce_next).  One `Call` object per function: called with integers, None and tensors in the declared positions it goes
 * straight to the library; anything else (keywords, other number types, wrong argument counts) goes to the Python function it was
 * made with, which says what is accepted and what is not.  A call through ctypes converts every argument through objects of its
 * own: 16 + 16 rows of 12 KB in one call take the host 4.2 us that way and 3.3 so (on a slower one 5.1 and 4.0), and the GPU 4.1.
 *
 * Built as the extension module paper_2406_03285_amd._calls; it is not linked to librb.so but given the functions' addresses,
 * so that it calls the library that the binding has loaded.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#define MAX_ARGS 10

typedef struct {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    uintptr_t address;          /* of the C function */
    char layout[MAX_ARGS + 1];  /* per argument: h - handle, p - device pointer, i - number (all 64 bits wide) */
    Py_ssize_t count;
    PyObject* general;          /* the Python function that takes everything */
    PyObject* dict;             /* attributes set on this object */
    PyObject* weakrefs;
} Call;

static PyObject* data_ptr_name;

/* 1: *out is set; 0: not one of the forms handled here (no exception pending); -1: the tensor's data_ptr() raised (the Python
   function takes its arguments in the same order and would raise the same; asked again there, an interrupt would be lost) */
static int plain_argument(PyObject* o, char kind, uint64_t* out)
{
    if (PyLong_CheckExact(o)) {
        *out = PyLong_AsUnsignedLongLongMask(o);        /* wraps like ctypes' 64-bit types do */
        return 1;
    }
    if (kind == 'i') return 0;
    if (o == Py_None) {
        *out = 0;
        return 1;
    }
    if (kind != 'p' || PyLong_Check(o)) return 0;       /* (bool and other kinds of int are no tensors) */
    PyObject* p = PyObject_CallMethodNoArgs(o, data_ptr_name);
    if (p == NULL) return -1;
    const int ok = PyLong_CheckExact(p);
    if (ok) *out = PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    return ok;
}

static PyObject* call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames)
{
    Call* c = (Call*)self;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf);
    uint64_t a[MAX_ARGS];
    int ok = n == c->count && (kwnames == NULL || PyTuple_GET_SIZE(kwnames) == 0);
    for (Py_ssize_t i = 0; ok > 0 && i < n; ++i) ok = plain_argument(args[i], c->layout[i], &a[i]);
    if (ok < 0) return NULL;
    if (ok == 0) return PyObject_Vectorcall(c->general, args, nargsf, kwnames);
    int status;
    Py_BEGIN_ALLOW_THREADS
    switch (n) {
    case 2: status = ((int (*)(uint64_t, uint64_t))c->address)(a[0], a[1]); break;
    case 6: status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(a[0], a[1], a[2], a[3], a[4], a[5]); break;
    case 7: status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(a[0], a[1], a[2], a[3], a[4], a[5], a[6]); break;
    default:
        status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(
            a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9]);
        break;
    }
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(status);
}

static int call_init(PyObject* self, PyObject* args, PyObject* kwargs)
{
    Call* c = (Call*)self;
    unsigned long long address;
    const char* layout;
    PyObject* general;
    if (kwargs != NULL && PyDict_GET_SIZE(kwargs) != 0) {
        PyErr_SetString(PyExc_TypeError, "Call takes no keywords");
        return -1;
    }
    if (!PyArg_ParseTuple(args, "KsO", &address, &layout, &general)) return -1;
    const size_t n = strlen(layout);
    if (address == 0 || (n != 2 && n != 6 && n != 7 && n != 10) || strspn(layout, "hpi") != n || !PyCallable_Check(general)) {
        PyErr_SetString(PyExc_ValueError, "Call(address, layout, general)");
        return -1;
    }
    c->address = (uintptr_t)address;
    memcpy(c->layout, layout, n + 1);
    c->count = (Py_ssize_t)n;
    Py_INCREF(general);
    Py_XSETREF(c->general, general);
    c->vectorcall = call;
    return 0;
}

static int call_traverse(PyObject* self, visitproc visit, void* arg)
{
    Py_VISIT(((Call*)self)->general);
    Py_VISIT(((Call*)self)->dict);
    return 0;
}

static int call_clear(PyObject* self)
{
    Py_CLEAR(((Call*)self)->general);
    Py_CLEAR(((Call*)self)->dict);
    return 0;
}

static void call_dealloc(PyObject* self)
{
    PyObject_GC_UnTrack(self);
    if (((Call*)self)->weakrefs != NULL) PyObject_ClearWeakRefs(self);
    call_clear(self);
    Py_TYPE(self)->tp_free(self);
}

/* __name__, __doc__, __wrapped__ (and with it inspect.signature) and the rest are the Python function's */
static PyObject* call_getattro(PyObject* self, PyObject* name)
{
    PyObject* v = PyObject_GenericGetAttr(self, name);
    Call* c = (Call*)self;
    if (v != NULL || c->general == NULL || !PyErr_ExceptionMatches(PyExc_AttributeError)) return v;
    PyErr_Clear();
    return PyObject_GetAttr(c->general, name);
}

static PyObject* call_wrapped(PyObject* self, void* unused)
{
    (void)unused;
    PyObject* g = ((Call*)self)->general;
    if (g == NULL) {            /* made without __init__ */
        PyErr_SetString(PyExc_AttributeError, "__wrapped__");
        return NULL;
    }
    Py_INCREF(g);
    return g;
}

/* What a Python function can do besides being called: it is copied and pickled as what its name stands for, ... */
static PyObject* call_reduce(PyObject* self, PyObject* unused)
{
    (void)unused;
    return PyObject_GetAttrString(self, "__qualname__");
}

/* ... becomes a method when it is an attribute of a class, ... */
static PyObject* call_descr_get(PyObject* self, PyObject* instance, PyObject* type)
{
    (void)type;
    if (instance == NULL || instance == Py_None) {
        Py_INCREF(self);
        return self;
    }
    return PyMethod_New(self, instance);
}

/* ... and has its own docstring */
static PyObject* call_doc(PyObject* self, void* unused)
{
    (void)unused;
    PyObject* g = ((Call*)self)->general;
    if (g == NULL) Py_RETURN_NONE;
    return PyObject_GetAttrString(g, "__doc__");
}

static PyMethodDef call_methods[] = {{"__reduce__", call_reduce, METH_NOARGS, NULL}, {NULL, NULL, 0, NULL}};
static PyGetSetDef call_getset[] = {
    {"__wrapped__", call_wrapped, NULL, NULL, NULL},
    {"__doc__", call_doc, NULL, NULL, NULL},
    {"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, NULL, NULL},
    {NULL, NULL, NULL, NULL, NULL},
};

static PyTypeObject CallType = {
    PyVarObject_HEAD_INIT(NULL, 0)
    .tp_name = "paper_2406_03285_amd._calls.Call",
    .tp_basicsize = sizeof(Call),
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_new = PyType_GenericNew,
    .tp_init = call_init,
    .tp_dealloc = call_dealloc,
    .tp_traverse = call_traverse,
    .tp_clear = call_clear,
    .tp_vectorcall_offset = offsetof(Call, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_getattro = call_getattro,
    .tp_setattro = PyObject_GenericSetAttr,
    .tp_descr_get = call_descr_get,
    .tp_dictoffset = offsetof(Call, dict),
    .tp_weaklistoffset = offsetof(Call, weakrefs),
    .tp_methods = call_methods,
    .tp_getset = call_getset,
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, NULL, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__calls(void)
{
    data_ptr_name = PyUnicode_InternFromString("data_ptr");
    if (data_ptr_name == NULL || PyType_Ready(&CallType) < 0) return NULL;
    PyObject* m = PyModule_Create(&module);
    if (m == NULL) return NULL;
    Py_INCREF(&CallType);
    if (PyModule_AddObject(m, "Call", (PyObject*)&CallType) < 0) {
        Py_DECREF(&CallType);
        Py_DECREF(m);
        return NULL;
    }
    return m;
}
