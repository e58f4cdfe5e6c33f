// Marshalling of the device entry points for Python, in native code: the module function of an entry point takes the
// arguments of the C function, with torch tensors (or None, or integer addresses) for its pointers, and returns its status.
//
// Why: with ctypes a call spends 0.3 us on each tensor in Python, 1.5 us (two tensors) to 4.7 us (sixteen) in
// all, more than the launch itself, and small decode steps are bound by the host.  Here it is 0.06 to 0.12 us.
//
// What this file does not know (other argument types, tensor subclasses, a failing tensor) goes to the Python
// function given to setup(), which marshals through ctypes: the same call, and the same exception where there is one.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <utility>

#include "../../include/infinigen.h"

namespace {

PyObject *through_ctypes = nullptr;      // f(name, *args)
PyTypeObject *desc_type = nullptr;       // the ctypes structure of ig_desc

enum Outcome { TAKEN, UNKNOWN, RAISED };

// one argument, by the type of the C parameter
template <typename T> Outcome take(PyObject *o, T **out) {
  if (o == Py_None) {
    *out = nullptr;
    return TAKEN;
  }
  if (THPVariable_CheckExact(o)) {
    try {
      const at::Tensor &t = THPVariable_Unpack(o);
      if (!t.is_contiguous()) {
        PyErr_SetString(PyExc_AssertionError, "tensors crossing the C ABI must be contiguous");
        return RAISED;
      }
      *out = static_cast<T *>(t.data_ptr());
      return TAKEN;
    } catch (...) {
      return UNKNOWN;
    }
  }
  if (PyLong_CheckExact(o)) {
    *out = reinterpret_cast<T *>((uintptr_t)PyLong_AsUnsignedLongLongMask(o));
    return PyErr_Occurred() ? RAISED : TAKEN;
  }
  return UNKNOWN;
}
Outcome take(PyObject *o, const ig_desc **out) {
  if (!PyObject_TypeCheck(o, desc_type)) return UNKNOWN;
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return UNKNOWN;
  }
  *out = static_cast<const ig_desc *>(b.buf);         // (the caller holds the structure for the length of the call)
  const bool whole = b.len == (Py_ssize_t)sizeof(ig_desc);
  PyBuffer_Release(&b);
  return whole ? TAKEN : UNKNOWN;
}
template <typename T> Outcome take_const(PyObject *o, const T **out) {
  T *p = nullptr;
  const Outcome got = take<T>(o, &p);
  *out = p;
  return got;
}
Outcome take(PyObject *o, const void **out) { return take_const<void>(o, out); }
Outcome take(PyObject *o, const float **out) { return take_const<float>(o, out); }
Outcome take(PyObject *o, const int32_t **out) { return take_const<int32_t>(o, out); }
Outcome take(PyObject *o, const ig_layer_io **out) { return take_const<ig_layer_io>(o, out); }
Outcome take(PyObject *o, const ig_buffer_set **out) { return take_const<ig_buffer_set>(o, out); }
Outcome take(PyObject *o, int *out) {
  if (!PyLong_CheckExact(o)) return UNKNOWN;
  *out = (int)PyLong_AsUnsignedLongMask(o);
  return PyErr_Occurred() ? RAISED : TAKEN;
}
Outcome take(PyObject *o, double *out) {
  if (!PyFloat_CheckExact(o)) return UNKNOWN;
  *out = PyFloat_AS_DOUBLE(o);
  return TAKEN;
}

PyObject *ask_python(const char *name, PyObject *const *args, Py_ssize_t n) {
  PyObject *all = PyTuple_New(n + 1);
  if (!all) return nullptr;
  PyObject *s = PyUnicode_FromString(name);
  if (!s) {
    Py_DECREF(all);
    return nullptr;
  }
  PyTuple_SET_ITEM(all, 0, s);
  for (Py_ssize_t i = 0; i < n; ++i) {
    Py_INCREF(args[i]);
    PyTuple_SET_ITEM(all, i + 1, args[i]);
  }
  PyObject *r = PyObject_Call(through_ctypes, all, nullptr);
  Py_DECREF(all);
  return r;
}

template <typename... A, size_t... I>
PyObject *run(const char *name, int (*f)(A...), PyObject *const *args, Py_ssize_t n, std::index_sequence<I...>) {
  if (!through_ctypes || n != (Py_ssize_t)sizeof...(A)) {
    if (through_ctypes) return ask_python(name, args, n);
    PyErr_SetString(PyExc_RuntimeError, "setup() has not been called");
    return nullptr;
  }
  std::tuple<A...> a;
  Outcome worst = TAKEN;
  auto each = [&](Outcome got) {
    if (got != TAKEN) worst = got;
    return got == TAKEN;
  };
  if (!(each(take(args[I], &std::get<I>(a))) && ...)) return worst == RAISED ? nullptr : ask_python(name, args, n);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f(std::get<I>(a)...);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}
template <typename... A> PyObject *run(const char *name, int (*f)(A...), PyObject *const *args, Py_ssize_t n) {
  return run(name, f, args, n, std::index_sequence_for<A...>{});
}

#define ENTRIES(X)                                                                                          \
  X(ig_wq_build) X(ig_slab_build) X(ig_append_token) X(ig_pool_touch) X(ig_pool_victim) X(ig_pool_replace)  \
  X(ig_pool_touch_policy) X(ig_pool_replace_policy) X(ig_speculate) X(ig_project) X(ig_scan_select)         \
  X(ig_project_indexed) X(ig_speculate_indexed) X(ig_speculate_equalized) X(ig_equalize_heads)              \
  X(ig_gather_kv) X(ig_sparse_attention) X(ig_sparse_attention_static) X(ig_sparse_attention_indexed)       \
  X(ig_gather_attention) X(ig_layer_step) X(ig_decode_step_overlapped) X(ig_skew_device)                    \
  X(ig_partial_index_device)

#define WRAPPER(NAME) \
  PyObject *call_##NAME(PyObject *, PyObject *const *args, Py_ssize_t n) { return run(#NAME, NAME, args, n); }
ENTRIES(WRAPPER)

PyObject *setup(PyObject *, PyObject *args) {
  PyObject *type, *f;
  if (!PyArg_ParseTuple(args, "O!O", &PyType_Type, &type, &f)) return nullptr;
  Py_INCREF(type);
  Py_INCREF(f);
  Py_XDECREF(reinterpret_cast<PyObject *>(desc_type));
  Py_XDECREF(through_ctypes);
  desc_type = reinterpret_cast<PyTypeObject *>(type);
  through_ctypes = f;
  Py_RETURN_NONE;
}

#define METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))call_##NAME, METH_FASTCALL, nullptr},
PyMethodDef methods[] = {{"setup", setup, METH_VARARGS, "setup(ctypes structure of ig_desc, f(name, *args))"},
                         ENTRIES(METHOD){nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ig_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch version whose tensor class this was compiled against, to be compared before any other use
PyMODINIT_FUNC PyInit__ig_call() {
  PyObject *m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "built_for", IG_BUILT_FOR) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
