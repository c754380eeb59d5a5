// The binding's tensor check in native code: a tensor's device address, after the same checks as binding.check_ptr, which is called
// for whatever does not pass (it raises, with the reason).  A call on a small batch names some twenty tensors, and four attributes
// of each looked up from Python took as long as the launches: a call of sf_classify 21.0 us on the host, with this 13.0 (9.4 in the library).
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

PyObject* slow_path = nullptr; // binding.check_ptr

// the address of a tensor that passes the checks, NULL without an error for anything else
PyObject* address(PyObject* t, PyObject* d)
{
    if (!THPVariable_CheckExact(t) || !(d == Py_None || THPDtype_Check(d))) return nullptr;
    try { // (no C++ exception may leave through Python; the other path says what it was)
        const at::Tensor& x = THPVariable_Unpack(t);
        if (x.is_cuda() && x.layout() == at::kStrided && x.is_contiguous() &&
            (d == Py_None || x.scalar_type() == reinterpret_cast<THPDtype*>(d)->scalar_type))
            return PyLong_FromVoidPtr(x.data_ptr());
    } catch (const std::exception&) {
    }
    return nullptr;
}

PyObject* checked(PyObject* const* args, Py_ssize_t n)
{
    PyObject* at = address(args[0], n == 2 ? args[1] : Py_None);
    return at || PyErr_Occurred() ? at : PyObject_Vectorcall(slow_path, args, (size_t)n, nullptr);
}

// ptr(tensor or None, dtype or nothing) -> the address as an int, None for None
PyObject* ptr(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n < 1 || n > 2) {
        PyErr_SetString(PyExc_TypeError, "ptr(tensor, dtype=None)");
        return nullptr;
    }
    if (args[0] == Py_None) Py_RETURN_NONE;
    return checked(args, n);
}

// need(tensor, dtype or nothing): the same for a tensor that may not be missing
PyObject* need(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n < 1 || n > 2 || args[0] == Py_None) {
        PyErr_SetString(PyExc_TypeError, n < 1 || n > 2 ? "need(tensor, dtype=None)" : "expected a tensor, got None");
        return nullptr;
    }
    return checked(args, n);
}

PyObject* set_slow_path(PyObject*, PyObject* f)
{
    Py_INCREF(f);
    Py_XSETREF(slow_path, f);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"ptr", (PyCFunction)(void (*)(void))ptr, METH_FASTCALL, "device address of a tensor, checked"},
    {"need", (PyCFunction)(void (*)(void))need, METH_FASTCALL, "the same, refusing None"},
    {"set_slow_path", set_slow_path, METH_O, "the function for tensors that do not pass the checks"},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
