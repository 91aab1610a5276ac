// The Python binding's way into the C boundary: takes the arguments of a binding function as they are, turns them into the plain
// values the boundary expects and calls it.  A small launch costs the host about as much in Python as in the HIP runtime
// when every argument passes through ctypes: append_kv 3.8 us a call without the
// boundary's own work, 1.0 through here (same host).
//
// A function is described by one letter per argument of the C function:
//   s  a ctypes structure of the given type, by address        p  device or host memory: an object with data_ptr(), an int, or None
//   i  a one-dimensional int32 numpy array, by address         N  that array's length (takes no argument)
//   n  an int                                                  t  a stream: an int, an object with cuda_stream, or None for torch's current one
// An argument in any other form makes the call return None without having called anything: the binding then goes the general way,
// which converts it or raises.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>

namespace {

constexpr int MAX_ARGS = 11;
// Integers and pointers only, so that one type serves all (arguments a function does not have are ignored by the calling convention).
typedef int (*CFunction)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t);

struct Bound {
    CFunction fn;
    char kinds[MAX_ARGS + 1];
    int n_args;                    // that the caller passes
    PyTypeObject *shape_type;
};

PyObject *g_data_ptr, *g_cuda_stream;                      // interned names
PyTypeObject *g_ndarray;
PyObject *g_get_device, *g_get_stream;                     // torch's, once it is in use

// An int object's value; false if it is none or does not fit.
bool int_value(PyObject *o, uint64_t *out) {
    if (!o || !PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow == 0) {
        *out = (uint64_t)v;
        return true;
    }
    *out = PyLong_AsUnsignedLongLong(o);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// ... of an int that a call or an attribute gave, which is dropped
bool take_int(PyObject *o, uint64_t *out) {
    if (!o) PyErr_Clear();
    const bool ok = int_value(o, out);
    Py_XDECREF(o);
    return ok;
}

PyObject *invoke(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
    const Bound *b = (const Bound *)PyCapsule_GetPointer(self, nullptr);
    if (!b) return nullptr;
    if (nargs != b->n_args) return PyErr_Format(PyExc_TypeError, "%d arguments, got %zd", b->n_args, nargs);
    uint64_t v[MAX_ARGS] = {};
    Py_buffer views[MAX_ARGS];
    int n_views = 0, next = 0;
    Py_ssize_t length = 0;
    bool ok = true;
    for (int i = 0; ok && b->kinds[i]; i++) {
        if (b->kinds[i] == 'N') {
            v[i] = (uint64_t)length;
            continue;
        }
        PyObject *a = args[next++];
        switch (b->kinds[i]) {
            case 's':
                ok = Py_TYPE(a) == b->shape_type && PyObject_GetBuffer(a, &views[n_views], PyBUF_SIMPLE) == 0;
                if (ok) v[i] = (uint64_t)(uintptr_t)views[n_views++].buf;
                break;
            case 'i':
                ok = Py_TYPE(a) == g_ndarray && PyObject_GetBuffer(a, &views[n_views], PyBUF_CONTIG_RO | PyBUF_FORMAT) == 0;
                if (ok) {
                    const Py_buffer &w = views[n_views++];
                    ok = w.ndim == 1 && w.itemsize == 4 && w.shape[0] > 0 && w.format && strcmp(w.format, "i") == 0;
                    length = w.ndim == 1 ? w.shape[0] : 0;
                    v[i] = (uint64_t)(uintptr_t)w.buf;
                }
                break;
            case 'n':
                ok = int_value(a, &v[i]);
                break;
            case 'p':
                if (a != Py_None && !int_value(a, &v[i])) ok = take_int(PyObject_CallMethodNoArgs(a, g_data_ptr), &v[i]);
                break;
            default:
                if (a == Py_None) {
                    PyObject *device = g_get_stream ? PyObject_CallNoArgs(g_get_device) : nullptr;
                    ok = device && take_int(PyObject_CallOneArg(g_get_stream, device), &v[i]);
                    Py_XDECREF(device);
                } else if (!int_value(a, &v[i])) {
                    ok = take_int(PyObject_GetAttr(a, g_cuda_stream), &v[i]);
                }
        }
        if (!ok) PyErr_Clear();
    }
    int rc = 0;
    if (ok) {
        Py_BEGIN_ALLOW_THREADS
        rc = b->fn(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10]);
        Py_END_ALLOW_THREADS
    }
    while (n_views > 0) PyBuffer_Release(&views[--n_views]);
    if (!ok) Py_RETURN_NONE;
    return PyLong_FromLong(rc);
}

PyMethodDef g_invoke = {"call", (PyCFunction)(void (*)(void))invoke, METH_FASTCALL, nullptr};

void drop_bound(PyObject *capsule) {
    Bound *b = (Bound *)PyCapsule_GetPointer(capsule, nullptr);
    if (!b) return;
    Py_XDECREF((PyObject *)b->shape_type);
    PyMem_Free(b);
}

// bind(address, kinds, type of the 's' argument) -> callable
PyObject *bind(PyObject *, PyObject *args) {
    unsigned long long address;
    const char *kinds;
    PyObject *type;
    if (!PyArg_ParseTuple(args, "KsO!", &address, &kinds, &PyType_Type, &type)) return nullptr;
    if (strlen(kinds) > MAX_ARGS || kinds[strspn(kinds, "spiNnt")]) return PyErr_Format(PyExc_ValueError, "kinds %s", kinds);
    Bound *b = (Bound *)PyMem_Calloc(1, sizeof(Bound));
    if (!b) return PyErr_NoMemory();
    b->fn = (CFunction)(uintptr_t)address;
    strcpy(b->kinds, kinds);
    for (const char *k = kinds; *k; k++) b->n_args += *k != 'N';
    Py_INCREF(type);
    b->shape_type = (PyTypeObject *)type;
    PyObject *capsule = PyCapsule_New(b, nullptr, drop_bound);
    if (!capsule) {
        Py_DECREF(type);
        PyMem_Free(b);
        return nullptr;
    }
    PyObject *call = PyCFunction_New(&g_invoke, capsule);
    Py_DECREF(capsule);
    return call;
}

// numpy(type of its arrays); torch(function for the current device, function for its current stream), or None and None: a call without a
// stream is left to the general way
PyObject *numpy(PyObject *, PyObject *type) {
    if (!PyType_Check(type)) return PyErr_Format(PyExc_TypeError, "a type");
    Py_INCREF(type);
    PyObject *old = (PyObject *)g_ndarray;
    g_ndarray = (PyTypeObject *)type;
    Py_XDECREF(old);
    Py_RETURN_NONE;
}

PyObject *torch(PyObject *, PyObject *args) {
    PyObject *device, *stream;
    if (!PyArg_ParseTuple(args, "OO", &device, &stream)) return nullptr;
    if (device == Py_None || stream == Py_None) device = stream = nullptr;
    Py_XINCREF(device);
    Py_XINCREF(stream);
    PyObject *old[] = {g_get_device, g_get_stream};
    g_get_device = device;
    g_get_stream = stream;
    Py_XDECREF(old[0]);
    Py_XDECREF(old[1]);
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {"numpy", numpy, METH_O, nullptr}, {"torch", torch, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
    g_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return g_data_ptr && g_cuda_stream ? PyModule_Create(&g_module) : nullptr;
}
