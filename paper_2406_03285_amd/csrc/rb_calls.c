/*
 * Native marshalling of the calls a training loop makes: rb_update, rb_sample_augment, rb_update_sample, rb_announce_next,
 * rb_update_sample_many, rb_announce_next_many, rb_pipeline_step_many and rb_pipeline_drain (rb_pipeline_step goes through ctypes).
 * One `Call` object per function: called with integers, None and tensors in the declared positions it goes straight to the library;
 * anything else (keywords, other number types, wrong argument counts) goes to the Python function it was made with, which says what is
 * accepted and what is not.  A call through ctypes converts every argument through objects of its own: 16 + 16 rows of 12 KB in one call
 * take the host 4.2 us that way and 3.3 so (on a slower one 5.1 and 4.0), and the GPU 4.1.
 * A call for many steps and its announcement make five arrays of pointers besides: for 20 steps through ctypes 28 us, which pipelines of
 * short steps wait for, and 4.3 so (16 steps of 21 + 7 rows of 44 KB on a stream of their own 54 -> 41 us a call).
 *
 * Built as the extension module paper_2406_03285_amd._calls; it is not linked to librb.so but given the functions' addresses,
 * so that it calls the library that the binding has loaded.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#define MAX_ARGS 12
#define MAX_STEPS 64            /* longer sequences go to the Python function */
#define MAX_SEQUENCES 4

typedef struct {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    uintptr_t address;          /* of the C function */
    char layout[MAX_ARGS + 1];  /* per argument: h - handle, p - device pointer, i - number (all 64 bits wide), v - list or tuple of as
                                   many device pointers as the number before the first of them says, s - stream (the last one, may be left out: null) */
    Py_ssize_t count;
    int rows;                   /* the C function has a further argument, an int64_t it sets: the call returns (status, that number) */
    PyObject* general;          /* the Python function that takes everything */
    PyObject* dict;             /* attributes set on this object */
    PyObject* weakrefs;
} Call;

static PyObject* data_ptr_name;
static PyObject* cuda_stream_name;

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

/* A list or tuple of `count` device pointers; results as above. */
static int pointer_sequence(PyObject* o, uint64_t count, uint64_t* out)
{
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return 0;
    if (count > MAX_STEPS) return 0;
    for (uint64_t i = 0; i < count; ++i) {
        /* (a tensor's data_ptr() may be anybody's code: the list is looked at anew and its item held) */
        if ((uint64_t)PySequence_Fast_GET_SIZE(o) != count) return 0;
        PyObject* item = PySequence_Fast_GET_ITEM(o, (Py_ssize_t)i);
        Py_INCREF(item);
        const int ok = plain_argument(item, 'p', &out[i]);
        Py_DECREF(item);
        if (ok <= 0) return ok;
    }
    return (uint64_t)PySequence_Fast_GET_SIZE(o) == count;
}

static int stream_argument(PyObject* o, uint64_t* out)
{
    if (o == Py_None || PyLong_Check(o)) return plain_argument(o, 'h', out);
    PyObject* p = PyObject_GetAttr(o, cuda_stream_name);
    if (p == NULL) return -1;
    const int ok = PyLong_CheckExact(p);
    if (ok) *out = PyLong_AsUnsignedLongLongMask(p);
    Py_DECREF(p);
    return ok;
}

static PyObject* call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames)
{
    Call* c = (Call*)self;
    const Py_ssize_t n = PyVectorcall_NARGS(nargsf), count = c->count;
    uint64_t a[MAX_ARGS + 1] = {0}, steps[MAX_SEQUENCES][MAX_STEPS], number = 0;
    int64_t rows = 0;
    int sequences = 0;
    int ok = (n == count || (n == count - 1 && c->layout[n] == 's')) && (kwnames == NULL || PyTuple_GET_SIZE(kwnames) == 0);
    for (Py_ssize_t i = 0; ok > 0 && i < n; ++i) {
        const char kind = c->layout[i];
        if (kind == 's') {
            ok = stream_argument(args[i], &a[i]);
        } else if (kind == 'v' && args[i] != Py_None) {
            ok = pointer_sequence(args[i], number, steps[sequences]);
            a[i] = (uint64_t)(uintptr_t)steps[sequences++];
        } else {
            ok = plain_argument(args[i], kind == 'v' ? 'h' : kind, &a[i]);
            if (kind == 'i' && sequences == 0) number = a[i];
        }
    }
    a[count] = (uint64_t)(uintptr_t)&rows;
    if (ok < 0) return NULL;
    if (ok == 0) return PyObject_Vectorcall(c->general, args, nargsf, kwnames);
    int status;
    Py_BEGIN_ALLOW_THREADS
    switch (count + c->rows) {
    case 2: status = ((int (*)(uint64_t, uint64_t))c->address)(a[0], a[1]); break;
    case 3: status = ((int (*)(uint64_t, uint64_t, uint64_t))c->address)(a[0], a[1], a[2]); break;
    case 6: status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(a[0], a[1], a[2], a[3], a[4], a[5]); break;
    case 7: status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(a[0], a[1], a[2], a[3], a[4], a[5], a[6]); break;
    case 10: status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9]); break;
    case 11: status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10]); break;
    default:
        status = ((int (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t))c->address)(
            a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12]);
        break;
    }
    Py_END_ALLOW_THREADS
    return c->rows ? Py_BuildValue("(iL)", status, (long long)rows) : PyLong_FromLong(status);
}

static int call_init(PyObject* self, PyObject* args, PyObject* kwargs)
{
    Call* c = (Call*)self;
    unsigned long long address;
    const char* layout;
    PyObject* general;
    int rows = 0;
    if (kwargs != NULL && PyDict_GET_SIZE(kwargs) != 0) {
        PyErr_SetString(PyExc_TypeError, "Call takes no keywords");
        return -1;
    }
    if (!PyArg_ParseTuple(args, "KsO|p", &address, &layout, &general, &rows)) return -1;
    const size_t n = strlen(layout), k = n + (size_t)rows;
    size_t sequences = 0;
    for (size_t i = 0; i < n; ++i) sequences += layout[i] == 'v';
    const char* stream = strchr(layout, 's');
    if (address == 0 || n > MAX_ARGS || (k != 2 && k != 3 && k != 6 && k != 7 && k != 10 && k != 11 && k != 13) || strspn(layout, "hpivs") != n ||
        sequences > MAX_SEQUENCES || (stream != NULL && stream != layout + n - 1) || !PyCallable_Check(general)) {
        PyErr_SetString(PyExc_ValueError, "Call(address, layout, general, rows=False)");
        return -1;
    }
    c->address = (uintptr_t)address;
    memcpy(c->layout, layout, n + 1);
    c->count = (Py_ssize_t)n;
    c->rows = rows;
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
    cuda_stream_name = PyUnicode_InternFromString("cuda_stream");
    if (data_ptr_name == NULL || cuda_stream_name == NULL || PyType_Ready(&CallType) < 0) return NULL;
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
