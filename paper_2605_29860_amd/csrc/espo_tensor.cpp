// The binding's check of one tensor argument, for Python: address(t, dtype, name, numel, shape).
//
// The C ABI takes bare pointers, so the binding looks at every tensor's type, layout and size first.  A call
// passes up to ten tensors, and from Python each look (dtype, is_contiguous, numel, shape, data_ptr) is a call
// of its own: 1.2 us per tensor on a slow host.  The same look takes 0.3 us here, the call from Python included.  With
// the current stream asked for its handle alone, us per call of a queue of calls, before -> now: espo_step on four
// rows 13.0 -> 10.0 (what the GPU takes), a four-row espo_advantages and espo_whiten 20.8 -> 13.3, espo_batch_stats
// 13.6 -> 10.0 (what the GPU takes).  Nothing is remembered between calls.
//
// And its calls of the library's functions: entry(name, address) is that function, taking the C function's arguments in
// order.  ctypes looks every argument's type up on each call, which took 1.4 of the 5 us that a call of ten arguments spends in the
// binding; here the conversions follow from the declarations in espo.h.  us per call of a queue of calls, before -> now: a four-row
// espo_advantages and espo_whiten 13.2 -> 11.1; in the binding alone, on another host: espo_advantages 3.5 -> 2.2, espo_step 7.5 -> 5.6.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string.h>

#include <tuple>
#include <type_traits>

#include "../../include/espo.h"
#include "../../include/espo_debug.h"

namespace {

// One argument of a C call.  Pointers: None, an address, or an object whose bytes are meant (a ctypes structure), which
// outlives the call.  Integers are taken modulo 2^64, floats rounded, as ctypes does it.
template <typename T>
bool from_python(PyObject* o, T& out) {
  if constexpr (std::is_pointer_v<T>) {
    if (o == Py_None) {
      out = nullptr;
    } else if (PyLong_Check(o)) {
      out = (T)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    } else {
      Py_buffer view;
      if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
      out = (T)view.buf;
      PyBuffer_Release(&view);
    }
  } else if constexpr (std::is_floating_point_v<T>) {
    out = (T)PyFloat_AsDouble(o);
  } else {
    out = (T)PyLong_AsUnsignedLongLongMask(o);
  }
  return !PyErr_Occurred();
}

template <typename... A, size_t... I>
bool all_from_python(PyObject* const* args, std::tuple<A...>& out, std::index_sequence<I...>) {
  return (from_python(args[I], std::get<I>(out)) && ...);
}

template <typename F>
struct Entry;
template <typename... A>
struct Entry<int(A...)> {
  static PyObject* call(PyObject* address, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != (Py_ssize_t)sizeof...(A)) {
      PyErr_Format(PyExc_TypeError, "need %zd arguments, got %zd", (Py_ssize_t)sizeof...(A), nargs);
      return nullptr;
    }
    std::tuple<A...> values;
    if (!all_from_python(args, values, std::index_sequence_for<A...>{})) return nullptr;
    const auto fn = (int (*)(A...))PyLong_AsVoidPtr(address);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = std::apply(fn, values);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  }
};

#define ESPO_ENTRY(name) {#name, (PyCFunction)(void (*)(void))Entry<decltype(::name)>::call, METH_FASTCALL, nullptr}
PyMethodDef entries[] = {ESPO_ENTRY(espo_step), ESPO_ENTRY(espo_debug_step), ESPO_ENTRY(espo_advantages), ESPO_ENTRY(espo_advantages_ws),
                         ESPO_ENTRY(espo_advantages_terminal), ESPO_ENTRY(espo_advantages_terminal_ws), ESPO_ENTRY(espo_advantages_packed),
                         ESPO_ENTRY(espo_length_order), ESPO_ENTRY(espo_whiten), ESPO_ENTRY(espo_whiten_from_ws),
                         ESPO_ENTRY(espo_batch_stats), ESPO_ENTRY(espo_batch_stats_static)};

// entry(name, address) -> the C function of that name at that address.
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  const char* name = nargs == 2 && PyLong_Check(args[1]) ? PyUnicode_AsUTF8(args[0]) : nullptr;
  if (name)
    for (PyMethodDef& def : entries)
      if (strcmp(def.ml_name, name) == 0) return PyCFunction_New(&def, args[1]);
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "entry(name, address)");
  return nullptr;
}

// address(t, dtype, name, numel or None, shape (a tuple) or None) -> int.  TypeError for another type or layout,
// ValueError for a tensor of fewer than `numel` elements or of another shape.  gpu_address: the same, and the tensor has to be on
// the GPU; None stays None.
template <bool Gpu>
PyObject* address(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  if (nargs != 5 || !THPDtype_Check(args[1])) {
    PyErr_SetString(PyExc_TypeError, "address(t, dtype, name, numel, shape)");
    return nullptr;
  }
  if (Gpu && args[0] == Py_None) Py_RETURN_NONE;
  if (!THPVariable_Check(args[0])) {
    PyErr_Format(PyExc_TypeError, "%U: need a contiguous GPU tensor of %S", args[2], args[1]);
    return nullptr;
  }
  const at::Tensor& t = THPVariable_Unpack(args[0]);
  if ((Gpu && !t.is_cuda()) || t.scalar_type() != ((THPDtype*)args[1])->scalar_type || !t.is_contiguous()) {
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

PyMethodDef methods[] = {{"address", (PyCFunction)(void (*)(void))address<false>, METH_FASTCALL, nullptr},
                         {"gpu_address", (PyCFunction)(void (*)(void))address<true>, METH_FASTCALL, nullptr},
                         {"entry", (PyCFunction)(void (*)(void))entry, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_espo_tensor", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__espo_tensor(void) { return PyModule_Create(&module); }
