// Python's way into disc_launch and disc_graph_launch: turns the argument lists of a call (dims,
// tensors, workspace) into the C arrays of the ABI.  Marshalling only, like the ctypes binding whose
// per-call part it is: with ctypes arrays a call spent 5 us here, more than a small kernel takes
// (37 x 768 fp32: 9.3 us a call, 4.4 us of them the kernel).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>

#include "disc.h"

namespace {

PyObject *s_data_ptr, *s_numel, *s_element_size;

// int(x) of any Python number, modulo 2^64
bool as_u64(PyObject* x, uint64_t* out) {
  if (PyLong_CheckExact(x)) {
    *out = PyLong_AsUnsignedLongLongMask(x);
    return !(*out == (uint64_t)-1 && PyErr_Occurred());
  }
  PyObject* n = PyNumber_Long(x);
  if (!n) return false;
  *out = PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  return !(*out == (uint64_t)-1 && PyErr_Occurred());
}

bool call_u64(PyObject* x, PyObject* method, uint64_t* out) {
  PyObject* r = PyObject_CallMethodNoArgs(x, method);
  if (!r) return false;
  const bool ok = as_u64(r, out);
  Py_DECREF(r);
  return ok;
}

// after a failed call_u64: the object has no such method (the error is cleared), or the method failed
bool lacks(PyObject* x, PyObject* method) {
  if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
  PyObject *type, *value, *trace;
  PyErr_Fetch(&type, &value, &trace);
  if (PyObject_HasAttr(x, method)) {
    PyErr_Restore(type, value, trace);
    return false;
  }
  Py_XDECREF(type);
  Py_XDECREF(value);
  Py_XDECREF(trace);
  return true;
}

// the device address of a tensor (anything with data_ptr()), or a raw address
bool as_address(PyObject* x, uint64_t* out) {
  if (PyLong_CheckExact(x)) return as_u64(x, out);
  if (call_u64(x, s_data_ptr, out)) return true;
  return lacks(x, s_data_ptr) && as_u64(x, out);
}

// A Python sequence as an array of 8-byte words; up to kInline of them need no allocation.
struct Words {
  static constexpr Py_ssize_t kInline = 24;
  uint64_t inl[kInline];
  uint64_t* p = inl;
  Py_ssize_t n = 0;
  ~Words() {
    if (p != inl) PyMem_Free(p);
  }
  bool fill(PyObject* seq, bool addresses) {
    PyObject* f = PySequence_Fast(seq, "expected a sequence");
    if (!f) return false;
    n = PySequence_Fast_GET_SIZE(f);
    if (n > kInline) p = (uint64_t*)PyMem_Malloc((size_t)n * sizeof(uint64_t));
    bool ok = p != nullptr;
    if (!ok) {
      p = inl;
      PyErr_NoMemory();
    }
    for (Py_ssize_t i = 0; ok && i < n; ++i) {
      // (the item is held: a data_ptr() written in Python could change the sequence)
      PyObject* x = PySequence_Fast_GET_ITEM(f, i);
      Py_INCREF(x);
      ok = addresses ? as_address(x, p + i) : as_u64(x, p + i);
      Py_DECREF(x);
      if (ok && PySequence_Fast_GET_SIZE(f) != n) {
        PyErr_SetString(PyExc_RuntimeError, "sequence changed size during the call");
        ok = false;
      }
    }
    Py_DECREF(f);
    return ok;
  }
};

typedef int (*launch_fn)(void*, int32_t, const int64_t*, int, const void* const*, int, void* const*, int, void*, size_t, void*);

// launch(function address, ctx address, id, dims, inputs, outputs, workspace or None, workspace
// bytes (0 or None: the size of the workspace tensor), stream) -> status.  The GIL is released during the call.
PyObject* launch(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  if (n_args != 9) {
    PyErr_SetString(PyExc_TypeError, "launch takes 9 arguments");
    return nullptr;
  }
  uint64_t fn, ctx, id, ws = 0, bytes = 0, stream;
  bool no_bytes = a[7] == Py_None;
  Words dims, ins, outs;
  if (!as_u64(a[0], &fn) || !as_u64(a[1], &ctx) || !as_u64(a[2], &id) || !dims.fill(a[3], false) || !ins.fill(a[4], true) ||
      !outs.fill(a[5], true) || (!no_bytes && !as_u64(a[7], &bytes)) || !as_u64(a[8], &stream))
    return nullptr;
  if (a[6] != Py_None) {
    if (!as_address(a[6], &ws)) return nullptr;
    if (bytes == 0 && !PyLong_CheckExact(a[6])) {
      uint64_t n = 0, size = 0;
      if (call_u64(a[6], s_numel, &n)) {
        if (!call_u64(a[6], s_element_size, &size)) return nullptr;
        bytes = n * size;
        no_bytes = false;
      } else if (!lacks(a[6], s_numel)) {
        return nullptr;
      }
    }
  }
  if (no_bytes) {
    PyErr_SetString(PyExc_TypeError, "workspace_bytes=None needs a workspace tensor to take the size from");
    return nullptr;
  }
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = reinterpret_cast<launch_fn>(fn)(reinterpret_cast<void*>(ctx), (int32_t)id, reinterpret_cast<const int64_t*>(dims.p), (int)dims.n,
                                       reinterpret_cast<const void* const*>(ins.p), (int)ins.n, reinterpret_cast<void* const*>(outs.p),
                                       (int)outs.n, reinterpret_cast<void*>(ws), (size_t)bytes, reinterpret_cast<void*>(stream));
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {{"launch", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(launch)), METH_FASTCALL,
                          "launch(fn, ctx, id, dims, inputs, outputs, workspace, workspace_bytes, stream) -> status"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pylaunch", "argument marshalling of disc_launch", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pylaunch() {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  if (!s_data_ptr || !s_numel || !s_element_size) return nullptr;
  return PyModule_Create(&module);
}
