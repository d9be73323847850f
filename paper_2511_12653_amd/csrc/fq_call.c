/* The calls of the binding that a program makes once per layer and step, without the interpreter's work on their
 * arguments.  A CPython extension: each function takes the descriptors, workspaces and streams that its Python
 * counterpart in binding.py takes; it recognises the forms below and leaves every other one, and every error, to
 * that counterpart, which `wrap` hands over.
 *
 *   descriptor   FqTensor / FqDistill itself (not a subclass)
 *   plan         ctypes.c_void_p
 *   workspace    torch.Tensor itself, or a tuple of two ints
 *   stream       left out: torch's current stream, once binding.py has given its lookups (`streams`)
 *
 * A launch costs the host 2.3 us in the runtime; what the interpreter and ctypes added to it came to 0.9 to 1.3 us.
 * As in ctypes, the interpreter's lock is free while the library runs.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/fq.h"

enum { FORWARD, BACKWARD, PLAN_RUN, PLAN_RUN_ADAM, DISTILL, LAYOUT_BYTES, CALLS };
static const char *const names[CALLS] = {"fq_forward", "fq_backward", "fq_plan_run", "fq_plan_run_adam", "fq_distill_loss",
                                         "fq_workspace_bytes"};

static PyObject *python_form[CALLS];                     /* the counterparts */
static PyObject *tensor_type, *distill_type, *pointer_type, *check;
static PyObject *raw_stream, *current_device, *torch_tensor;
static PyObject *str_data_ptr, *str_numel, *str_element_size;

static PyObject *to_python(int call, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    if (!python_form[call]) {
        PyErr_Format(PyExc_RuntimeError, "%s has no Python form yet", names[call]);
        return NULL;
    }
    return PyObject_Vectorcall(python_form[call], args, (size_t)nargs, kwnames);
}

static int is_a(PyObject *o, PyObject *type) { return (PyObject *)Py_TYPE(o) == type; }

/* Address of a ctypes object's memory; the caller's reference keeps it there. */
static void *memory_of(PyObject *o)
{
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return NULL;
    void *p = view.buf;
    PyBuffer_Release(&view);
    return p;
}

static int current_stream(void **stream)
{
    PyObject *device = PyObject_CallNoArgs(current_device);
    if (!device) return -1;
    PyObject *handle = PyObject_CallOneArg(raw_stream, device);
    Py_DECREF(device);
    if (!handle) return -1;
    *stream = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    return *stream == NULL && PyErr_Occurred() ? -1 : 0;
}

static int method_value(PyObject *o, PyObject *name, size_t *value)
{
    PyObject *v = PyObject_CallMethodNoArgs(o, name);
    if (!v) return -1;
    *value = PyLong_AsSize_t(v);
    Py_DECREF(v);
    return *value == (size_t)-1 && PyErr_Occurred() ? -1 : 0;
}

static int is_workspace(PyObject *o)
{
    return is_a(o, torch_tensor) || (PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2 &&
                                     PyLong_CheckExact(PyTuple_GET_ITEM(o, 0)) && PyLong_CheckExact(PyTuple_GET_ITEM(o, 1)));
}

/* 0, -1 with an exception set, or 1: an integer that a pointer or a size_t does not hold.  ctypes takes those (it
 * drops the upper bits), so they are left to the Python form. */
static int workspace(PyObject *o, void **p, size_t *bytes)
{
    if (PyTuple_CheckExact(o)) {
        *p = PyLong_AsVoidPtr(PyTuple_GET_ITEM(o, 0));
        if (*p != NULL || !PyErr_Occurred()) *bytes = PyLong_AsSize_t(PyTuple_GET_ITEM(o, 1));
        if (!PyErr_Occurred()) return 0;
        if (!PyErr_ExceptionMatches(PyExc_OverflowError)) return -1;
        PyErr_Clear();
        return 1;
    }
    size_t address, count, each;
    if (method_value(o, str_data_ptr, &address) || method_value(o, str_numel, &count) || method_value(o, str_element_size, &each))
        return -1;
    *p = (void *)address;
    *bytes = count * each;
    return 0;
}

static PyObject *done(fq_status status)
{
    if (status == FQ_OK) Py_RETURN_NONE;
    return PyObject_CallFunction(check, "i", (int)status);       /* raises FqError */
}

static PyObject *call_forward(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    if (nargs != 1 || kwnames || !raw_stream || !is_a(args[0], tensor_type)) return to_python(FORWARD, args, nargs, kwnames);
    const fq_tensor *t = memory_of(args[0]);
    void *stream;
    fq_status status;
    if (!t || current_stream(&stream)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    status = fq_forward(t, stream);
    Py_END_ALLOW_THREADS
    return done(status);
}

static PyObject *call_backward(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    if (nargs != 2 || kwnames || !raw_stream || !is_a(args[0], tensor_type) || !is_workspace(args[1]))
        return to_python(BACKWARD, args, nargs, kwnames);
    const fq_tensor *t = memory_of(args[0]);
    void *stream, *ws;
    size_t bytes;
    fq_status status;
    if (!t) return NULL;
    const int left = workspace(args[1], &ws, &bytes);
    if (left > 0) return to_python(BACKWARD, args, nargs, kwnames);
    if (left || current_stream(&stream)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    status = fq_backward(t, ws, bytes, stream);
    Py_END_ALLOW_THREADS
    return done(status);
}

static PyObject *call_distill(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    if (nargs != 2 || kwnames || !raw_stream || !is_a(args[0], distill_type) || !is_workspace(args[1]))
        return to_python(DISTILL, args, nargs, kwnames);
    const fq_distill *d = memory_of(args[0]);
    void *stream, *ws;
    size_t bytes;
    fq_status status;
    if (!d) return NULL;
    const int left = workspace(args[1], &ws, &bytes);
    if (left > 0) return to_python(DISTILL, args, nargs, kwnames);
    if (left || current_stream(&stream)) return NULL;
    Py_BEGIN_ALLOW_THREADS
    status = fq_distill_loss(d, ws, bytes, stream);
    Py_END_ALLOW_THREADS
    return done(status);
}

static PyObject *call_plan_run(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    if (nargs != 1 || kwnames || !raw_stream || !is_a(args[0], pointer_type)) return to_python(PLAN_RUN, args, nargs, kwnames);
    void **plan = memory_of(args[0]);
    void *stream;
    fq_status status;
    if (!plan || current_stream(&stream)) return NULL;
    const fq_plan *p = *plan;
    Py_BEGIN_ALLOW_THREADS
    status = fq_plan_run(p, stream);
    Py_END_ALLOW_THREADS
    return done(status);
}

static PyObject *call_plan_run_adam(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    if (nargs != 2 || kwnames || !raw_stream || !is_a(args[0], pointer_type) || !PyLong_CheckExact(args[1]))
        return to_python(PLAN_RUN_ADAM, args, nargs, kwnames);
    int overflow;
    const long long step = PyLong_AsLongLongAndOverflow(args[1], &overflow);
    if (overflow) return to_python(PLAN_RUN_ADAM, args, nargs, kwnames);
    void **plan = memory_of(args[0]);
    void *stream;
    fq_status status;
    if (!plan || current_stream(&stream)) return NULL;
    fq_plan *p = *plan;
    Py_BEGIN_ALLOW_THREADS
    status = fq_plan_run_adam(p, step, stream);
    Py_END_ALLOW_THREADS
    return done(status);
}

static PyObject *call_workspace_bytes(PyObject *self, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames)
{
    (void)self;
    if (nargs != 2 || kwnames || !tensor_type || !is_a(args[0], tensor_type) || !PyLong_CheckExact(args[1]))
        return to_python(LAYOUT_BYTES, args, nargs, kwnames);
    const fq_tensor *t = memory_of(args[0]);
    if (!t) return NULL;
    int overflow;
    const long mode = PyLong_AsLongAndOverflow(args[1], &overflow);
    if (overflow || mode != (int)mode) return to_python(LAYOUT_BYTES, args, nargs, kwnames);
    return PyLong_FromSize_t(fq_workspace_bytes(t, 1, (int)mode));
}

static void keep(PyObject **slot, PyObject *value)
{
    PyObject *old = *slot;
    Py_XINCREF(value);
    *slot = value;
    Py_XDECREF(old);
}

static PyObject *setup(PyObject *self, PyObject *args)
{
    PyObject *t, *d, *p, *c;
    (void)self;
    if (!PyArg_ParseTuple(args, "OOOO", &t, &d, &p, &c)) return NULL;
    keep(&tensor_type, t);
    keep(&distill_type, d);
    keep(&pointer_type, p);
    keep(&check, c);
    Py_RETURN_NONE;
}

static PyObject *streams(PyObject *self, PyObject *args)
{
    PyObject *raw, *device, *tensor;
    (void)self;
    if (!PyArg_ParseTuple(args, "OOO", &raw, &device, &tensor)) return NULL;
    keep(&torch_tensor, tensor);
    keep(&current_device, device);
    keep(&raw_stream, raw);
    Py_RETURN_NONE;
}

static PyObject *wrap(PyObject *self, PyObject *function)
{
    PyObject *name = PyObject_GetAttrString(function, "__name__");
    if (!name) return NULL;
    for (int i = 0; i < CALLS; ++i) {
        if (PyUnicode_CompareWithASCIIString(name, names[i]) == 0) {
            keep(&python_form[i], function);
            Py_DECREF(name);
            return PyObject_GetAttrString(self, names[i]);
        }
    }
    PyErr_Format(PyExc_ValueError, "no native form of %U", name);
    Py_DECREF(name);
    return NULL;
}

#define FAST(f) (PyCFunction)(void (*)(void)) f, METH_FASTCALL | METH_KEYWORDS
static PyMethodDef methods[] = {
    {"fq_forward", FAST(call_forward), "fq_forward(t, stream=None)\n--\n\n"},
    {"fq_backward", FAST(call_backward), "fq_backward(t, workspace, stream=None)\n--\n\n"},
    {"fq_plan_run", FAST(call_plan_run), "fq_plan_run(plan, stream=None)\n--\n\n"},
    {"fq_plan_run_adam", FAST(call_plan_run_adam), "fq_plan_run_adam(plan, step, stream=None)\n--\n\n"},
    {"fq_distill_loss", FAST(call_distill), "fq_distill_loss(d, workspace, stream=None)\n--\n\n"},
    {"fq_workspace_bytes", FAST(call_workspace_bytes), "fq_workspace_bytes(tensors, mode)\n--\n\n"},
    {"setup", setup, METH_VARARGS, "setup(FqTensor, FqDistill, c_void_p, check)\n--\n\n"},
    {"streams", streams, METH_VARARGS, "streams(raw, device, Tensor)\n--\n\n"},
    {"wrap", wrap, METH_O, "wrap(function)\n--\n\nThe native form of the binding's function, which takes what that one leaves to it."},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fqcall", "The binding's calls per layer and step.", -1, methods,
                                    NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fqcall(void)
{
    str_data_ptr = PyUnicode_InternFromString("data_ptr");
    str_numel = PyUnicode_InternFromString("numel");
    str_element_size = PyUnicode_InternFromString("element_size");
    if (!str_data_ptr || !str_numel || !str_element_size) return NULL;
    return PyModule_Create(&module);
}
