// The per-call part of the Python binding in native code: check the tensors
// of a call, collect their addresses and make the C call.
//
// Checked one attribute at a time from Python, the sixteen tensors of an
// eight-rank call cost 7-10 us, several times what the launch and the
// collective itself take at small sizes.  Here a call's tensors are checked in
// well under a microsecond.
//
// call(fn, first, send, recv, n, send_numel, recv_numel, bf16, stream): fn is
// the address of a library function (first, send, recv, stream) -> status, or,
// with recv = None, (first, send, stream) -> status.  Returns the status, or -1
// without calling fn when a tensor is not plainly right (another class,
// device, layout, type, size, or not contiguous, or without storage): the
// caller then takes the checks in Python, which accept or raise.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>

namespace {

constexpr Py_ssize_t kMaxRanks = 16;

// Addresses of the tensors of a list or tuple; false if any needs a closer look.
bool collect(PyObject *seq, Py_ssize_t n, int64_t numel, at::ScalarType type, void **out)
{
    if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) return false;
    if (PySequence_Fast_GET_SIZE(seq) != n) return false;
    PyObject **items = PySequence_Fast_ITEMS(seq);
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject *o = items[i];
        // Subclasses may answer for themselves (__torch_function__).
        if (!THPVariable_CheckExact(o) && (PyObject *)Py_TYPE(o) != ParameterClass) return false;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != type ||
            t.numel() != numel || !t.has_storage() || !t.is_contiguous())
            return false;
        out[i] = t.data_ptr();
    }
    return true;
}

PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 9) {
        PyErr_SetString(PyExc_TypeError, "call takes 9 arguments");
        return nullptr;
    }
    void *fn = PyLong_AsVoidPtr(args[0]), *first = PyLong_AsVoidPtr(args[1]), *stream = PyLong_AsVoidPtr(args[8]);
    const Py_ssize_t n = PyLong_AsSsize_t(args[4]);
    const int64_t send_numel = PyLong_AsLongLong(args[5]), recv_numel = PyLong_AsLongLong(args[6]);
    const long bf16 = PyLong_AsLong(args[7]);
    if (PyErr_Occurred()) return nullptr;
    if (!fn || n < 1 || n > kMaxRanks) return PyLong_FromLong(-1);
    const bool in_place = args[3] == Py_None;
    void *send[kMaxRanks], *recv[kMaxRanks];
    try {
        const at::ScalarType type = bf16 ? at::kBFloat16 : at::kFloat;
        if (!collect(args[2], n, send_numel, type, send)) return PyLong_FromLong(-1);
        if (!in_place && !collect(args[3], n, recv_numel, type, recv)) return PyLong_FromLong(-1);
    } catch (...) {
        return PyLong_FromLong(-1);  // the checks in Python raise what there is to raise
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (in_place) rc = ((int (*)(void *, void **, void *))fn)(first, send, stream);
    else rc = ((int (*)(void *, void **, void **, void *))fn)(first, send, recv, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// call_bound(fn, first, send, recv, stream): the same for addresses that were
// collected before; recv = 0 for the functions without it.
PyObject *call_bound(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "call_bound takes 5 arguments");
        return nullptr;
    }
    void *fn = PyLong_AsVoidPtr(args[0]), *first = PyLong_AsVoidPtr(args[1]), *stream = PyLong_AsVoidPtr(args[4]);
    void **send = (void **)PyLong_AsVoidPtr(args[2]), **recv = (void **)PyLong_AsVoidPtr(args[3]);
    if (PyErr_Occurred()) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    if (!recv) rc = ((int (*)(void *, void **, void *))fn)(first, send, stream);
    else rc = ((int (*)(void *, void **, void **, void *))fn)(first, send, recv, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"call_bound", (PyCFunction)(void (*)(void))call_bound, METH_FASTCALL, "Make the C call on collected addresses."},
    {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "Check the tensors and make the C call."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tensor_args", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the torch whose headers this was compiled with.  The binding
// uses the module with that one alone.
PyMODINIT_FUNC PyInit__tensor_args(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", AR_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
