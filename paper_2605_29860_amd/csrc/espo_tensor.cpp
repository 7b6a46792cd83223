// The binding's check of one tensor argument, for Python: address(t, dtype, name, numel, shape).
//
// The C ABI takes bare pointers, so the binding looks at every tensor's type, layout and size first.  A call
// passes up to ten tensors, and from Python each look (dtype, is_contiguous, numel, shape, data_ptr) is a call
// of its own: 1.2 us per tensor on a slow host.  The same look takes 0.3 us here, the call from Python included.  With
// the current stream asked for its handle alone, us per call of a queue of calls, before -> now: espo_step on four
// rows 13.0 -> 10.0 (what the GPU takes), a four-row espo_advantages and espo_whiten 20.8 -> 13.3, espo_batch_stats
// 13.6 -> 10.0 (what the GPU takes).  Nothing is remembered between calls.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

// address(t, dtype, name, numel or None, shape (a tuple) or None) -> int.  TypeError for another type or layout,
// ValueError for a tensor of fewer than `numel` elements or of another shape.
PyObject* address(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 5 || !THPDtype_Check(args[1])) {
    PyErr_SetString(PyExc_TypeError, "address(t, dtype, name, numel, shape)");
    return nullptr;
  }
  if (!THPVariable_Check(args[0])) {
    PyErr_Format(PyExc_TypeError, "%U: need a contiguous GPU tensor of %S", args[2], args[1]);
    return nullptr;
  }
  const at::Tensor& t = THPVariable_Unpack(args[0]);
  if (t.scalar_type() != ((THPDtype*)args[1])->scalar_type || !t.is_contiguous()) {
    PyErr_Format(PyExc_TypeError, "%U: need a contiguous GPU tensor of %S", args[2], args[1]);
    return nullptr;
  }
  if (args[3] != Py_None) {
    const long long need = PyLong_AsLongLong(args[3]);
    if (need == -1 && PyErr_Occurred()) return nullptr;
    if (t.numel() < need) {
      PyErr_Format(PyExc_ValueError, "%U: need at least %lld elements, got %lld", args[2], need, (long long)t.numel());
      return nullptr;
    }
  }
  if (args[4] != Py_None) {
    const auto sizes = t.sizes();
    bool same = PyTuple_Check(args[4]) && PyTuple_GET_SIZE(args[4]) == (Py_ssize_t)sizes.size();
    for (size_t i = 0; same && i < sizes.size(); ++i) {
      const long long n = PyLong_AsLongLong(PyTuple_GET_ITEM(args[4], (Py_ssize_t)i));
      if (n == -1 && PyErr_Occurred()) return nullptr;
      same = n == sizes[i];
    }
    if (!same) {
      PyObject* got = PyTuple_New((Py_ssize_t)sizes.size());
      if (!got) return nullptr;
      for (size_t i = 0; i < sizes.size(); ++i) PyTuple_SET_ITEM(got, (Py_ssize_t)i, PyLong_FromLongLong(sizes[i]));
      PyErr_Format(PyExc_ValueError, "%U: need shape %S, got %S", args[2], args[4], got);
      Py_DECREF(got);
      return nullptr;
    }
  }
  return PyLong_FromVoidPtr(t.data_ptr());
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"address", (PyCFunction)(void (*)(void))address, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_espo_tensor", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__espo_tensor(void) { return PyModule_Create(&module); }
