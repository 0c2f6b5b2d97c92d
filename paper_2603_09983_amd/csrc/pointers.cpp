// Device addresses of a call's tensors for the Python binding, read in one call from Python.  Argument by argument in Python,
// three attribute calls each, that was half of the host time of a call (24 layers' cache plan: 2.7 of 5.6 us), which bounds the
// control loop's three short launches.  Only what needs no second look is answered here: a plain torch.Tensor or Parameter in
// device memory, contiguous.  For anything else the binding's own function decides, and raises what it raises.
//
// Reads torch's own objects through its C++ headers: good for the torch that it was compiled against and no other, so the
// module says which one that was and the binding asks before it calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

PyObject *g_general = nullptr;   // the binding's function for one tensor

PyObject *address(PyObject *o)
{
    if (o == Py_None) {
        Py_INCREF(Py_None);
        return Py_None;
    }
    if (THPVariable_CheckExact(o)) {
        try {
            const at::Tensor &t = THPVariable_Unpack(o);
            if (t.is_cuda() && t.is_contiguous()) return PyLong_FromVoidPtr(t.data_ptr());
        } catch (...) {
            // (a tensor without storage or strides of its own: the general function says what is wrong with it)
        }
    }
    return PyObject_CallOneArg(g_general, o);
}

// pointers(*tensors) -> tuple of addresses (None stays None)
PyObject *pointers(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (!g_general) {
        PyErr_SetString(PyExc_RuntimeError, "general() has not been called");
        return nullptr;
    }
    PyObject *out = PyTuple_New(n);
    for (Py_ssize_t i = 0; out && i < n; ++i) {
        PyObject *p = address(args[i]);
        if (!p) {
            Py_DECREF(out);
            return nullptr;
        }
        PyTuple_SET_ITEM(out, i, p);
    }
    return out;
}

// general(f): f(tensor) gives the address of what pointers() does not answer itself
PyObject *general(PyObject *, PyObject *f)
{
    Py_INCREF(f);
    Py_XDECREF(g_general);
    g_general = f;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"pointers", (PyCFunction)(void (*)(void))pointers, METH_FASTCALL, "addresses of device-resident contiguous tensors"},
    {"general", general, METH_O, "the function for anything else"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pointers", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pointers(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_build", MOE_TORCH_BUILD) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
