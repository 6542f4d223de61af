// Device pointers of the binding's tensor arguments, with the checks that go with them.
//
// A join of 32 queries is 22 us, 10 of them on the device.  Its seven tensors cost 0.28 us each when
// their dtype, device, layout and address are asked for one after the other through the interpreter,
// 0.09 here: 21.7 -> 20.3 us a call.
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

PyObject* in_python = nullptr;  // the same in Python, for everything that is not a plain tensor as it should be

// ptr(tensor or None, dtype, what): the tensor's address, None for None.
PyObject* ptr(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n == 3) {
        if (args[0] == Py_None) Py_RETURN_NONE;
        // (subclasses, and any tensor while a torch function mode is on, keep their say)
        if (THPVariable_CheckExact(args[0]) && THPDtype_Check(args[1]) &&
            !at::impl::torch_function_mode_enabled()) {
            const at::Tensor& t = THPVariable_Unpack(args[0]);
            if (t.scalar_type() == reinterpret_cast<THPDtype*>(args[1])->scalar_type && t.is_cuda() &&
                t.is_contiguous())
                return PyLong_FromVoidPtr(t.data_ptr());
        }
    }
    if (in_python == nullptr) {
        PyErr_SetString(PyExc_RuntimeError, "otherwise() has not been called");
        return nullptr;
    }
    return PyObject_Vectorcall(in_python, args, (size_t)n, nullptr);
    END_HANDLE_TH_ERRORS
}

// otherwise(function): what ptr calls for arguments that it does not handle itself.
PyObject* otherwise(PyObject*, PyObject* function) {
    PyObject* before = in_python;
    Py_INCREF(function);
    in_python = function;
    Py_XDECREF(before);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"ptr", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(ptr)), METH_FASTCALL, nullptr},
    {"otherwise", otherwise, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr,
                      nullptr};

}  // namespace

// built_for: the torch and the Python whose headers this was compiled with; with others it must not be used.
PyMODINIT_FUNC PyInit__marshal() {
    PyObject* m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", SUREL_TORCH_VERSION " " PY_VERSION) != 0)
        Py_CLEAR(m);
    return m;
}
