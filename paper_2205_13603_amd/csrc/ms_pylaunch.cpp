// CPython entry to ms_variant_launch.  A launch of a small operator costs the host more than the device: marshalling its
// pointers through ctypes objects took 1.7 of 4.5 us a call.  The address of ms_variant_launch comes from the binding,
// which loads libms.so once and in its own order; nothing here links to it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

namespace {

typedef int32_t (*launch_fn)(void *variant, const void *const *inputs, void *const *outputs, void *workspace, int32_t instances, void *stream);
launch_fn g_launch = nullptr;

// a device pointer: an int, None for a null pointer, or a ctypes pointer holding one of them
bool pointer(PyObject *o, void **out, bool held = false)
{
    *out = nullptr;
    if (o == Py_None) return true;
    if (!PyLong_Check(o)) {
        PyObject *v = held ? nullptr : PyObject_GetAttrString(o, "value");
        const bool ok = v && pointer(v, out, true);
        Py_XDECREF(v);
        if (!ok) PyErr_Format(PyExc_TypeError, "a device pointer is an int or None, not %.100s", Py_TYPE(o)->tp_name);
        return ok;
    }
    *out = PyLong_AsVoidPtr(o);
    return *out != nullptr || !PyErr_Occurred();
}

PyObject *bind(PyObject *, PyObject *address)
{
    void *p = nullptr;
    if (!pointer(address, &p)) return nullptr;
    g_launch = reinterpret_cast<launch_fn>(p);
    Py_RETURN_NONE;
}

// launch(variant, inputs, output, instances, stream, workspace) -> status code
PyObject *launch(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 6 || !g_launch) {
        PyErr_SetString(PyExc_TypeError, "launch(variant, inputs, output, instances, stream, workspace) after bind()");
        return nullptr;
    }
    void *variant, *in[4] = {nullptr, nullptr, nullptr, nullptr}, *out, *stream, *workspace;
    PyObject *seq = PySequence_Fast(args[1], "inputs: a sequence of device pointers");
    if (!seq) return nullptr;
    const Py_ssize_t count = PySequence_Fast_GET_SIZE(seq);
    bool ok = count <= 4;
    if (!ok) PyErr_Format(PyExc_ValueError, "%zd inputs, an operator has at most 4", count);
    for (Py_ssize_t i = 0; ok && i < count; ++i) ok = pointer(PySequence_Fast_GET_ITEM(seq, i), &in[i]);
    Py_DECREF(seq);
    if (!ok || !pointer(args[0], &variant) || !pointer(args[2], &out) || !pointer(args[4], &stream) || !pointer(args[5], &workspace)) return nullptr;
    const int32_t instances = (int32_t)PyLong_AsUnsignedLongMask(args[3]);
    if (PyErr_Occurred()) return nullptr;
    int32_t rc;
    Py_BEGIN_ALLOW_THREADS // the queue of a stream may be full
    rc = g_launch(variant, in, &out, workspace, instances, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {{"bind", bind, METH_O, "address of ms_variant_launch"},
                         {"launch", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(launch)), METH_FASTCALL, "one launch, returns the status code"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_launch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__launch(void) { return PyModule_Create(&module); }
