// What binding.py does once per tensor argument and once per call, without the interpreter: checks and the address of a tensor, and torch's current stream.
//   ptr(tensor or None, dtype or None) -> address or None; the checks and errors of binding._ptr_any, which serves everything that is not a plain tensor
//   stream() -> the current stream of the current device
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

PyObject* g_any = nullptr;                            // binding._ptr_any

PyObject* ptr(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n < 1 || n > 2) {
        PyErr_SetString(PyExc_TypeError, "ptr(tensor, dtype=None)");
        return nullptr;
    }
    PyObject* t = args[0];
    PyObject* dtype = n == 2 ? args[1] : Py_None;
    if (t == Py_None) Py_RETURN_NONE;
    if (THPVariable_CheckExact(t) && (dtype == Py_None || THPDtype_Check(dtype))) {
        const at::Tensor& x = THPVariable_Unpack(t);
        if (x.is_cuda() && x.is_contiguous() && (dtype == Py_None || x.scalar_type() == reinterpret_cast<THPDtype*>(dtype)->scalar_type))
            return PyLong_FromVoidPtr(x.data_ptr());
    }
    return PyObject_CallFunctionObjArgs(g_any, t, dtype, nullptr);
    END_HANDLE_TH_ERRORS
}

PyObject* stream(PyObject*, PyObject*)
{
    HANDLE_TH_ERRORS
    return PyLong_FromVoidPtr(c10::hip::getCurrentHIPStream().stream());
    END_HANDLE_TH_ERRORS
}

PyObject* set_any(PyObject*, PyObject* f)
{
    Py_INCREF(f);
    Py_XSETREF(g_any, f);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"ptr", (PyCFunction)(void (*)(void))ptr, METH_FASTCALL, nullptr},
                         {"stream", stream, METH_NOARGS, nullptr},
                         {"set_any", set_any, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
