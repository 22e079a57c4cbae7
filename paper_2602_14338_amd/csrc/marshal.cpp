// Checks and device pointers of a call's tensors in one step: the part of the binding that costs most of a small
// call when it runs in Python (fifteen tensors at 0.5 us each against 3 us for a launch).
//
//   pointers(t0, dtype0, name0, t1, dtype1, name1, ...) -> (address or None, ...)
//
// Per tensor, in this order: None stays None; it must live on the GPU, have the dtype (None: any) and be
// contiguous.  Anything but a plain tensor or parameter goes to the Python function given to setup(), which
// performs the same checks.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

namespace {

PyObject* g_error = nullptr;      // exception class of the binding
PyObject* g_general = nullptr;    // pointer of any other kind of tensor: f(t, dtype, name)

PyObject* setup(PyObject*, PyObject* args) {
  PyObject *error, *general;
  if (!PyArg_ParseTuple(args, "OO", &error, &general)) return nullptr;
  Py_INCREF(error);
  Py_INCREF(general);
  Py_XSETREF(g_error, error);
  Py_XSETREF(g_general, general);
  Py_RETURN_NONE;
}

PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (!g_error || n_args % 3 != 0) {
    PyErr_SetString(PyExc_TypeError, "pointers: expected (tensor, dtype, name) triples after setup()");
    return nullptr;
  }
  THPObjectPtr out(PyTuple_New(n_args / 3));
  if (!out) return nullptr;
  for (Py_ssize_t i = 0; i < n_args; i += 3) {
    PyObject *t = args[i], *dtype = args[i + 1], *name = args[i + 2], *value;
    if (t == Py_None) {
      value = Py_NewRef(Py_None);
    } else if (!THPVariable_CheckExact(t)) {
      value = PyObject_CallFunctionObjArgs(g_general, t, dtype, name, nullptr);
    } else {
      const at::Tensor& x = THPVariable_Unpack(t);
      if (!x.is_cuda()) {
        PyErr_Format(g_error, "%U: expected a GPU tensor", name);
        return nullptr;
      }
      if (dtype != Py_None && x.scalar_type() != reinterpret_cast<THPDtype*>(dtype)->scalar_type) {
        THPObjectPtr got(PyObject_GetAttrString(t, "dtype"));
        if (got) PyErr_Format(g_error, "%U: expected dtype %S, got %S", name, dtype, got.get());
        return nullptr;
      }
      if (!x.is_contiguous()) {
        PyErr_Format(g_error, "%U: expected a contiguous tensor", name);
        return nullptr;
      }
      value = PyLong_FromVoidPtr(x.data_ptr());
    }
    if (!value) return nullptr;
    PyTuple_SET_ITEM(out.get(), i / 3, value);
  }
  return out.release();
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, "setup(error class, pointer function for other kinds of tensors)"},
    {"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pointers)), METH_FASTCALL,
     "pointers(t0, dtype0, name0, ...) -> tuple of addresses"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
