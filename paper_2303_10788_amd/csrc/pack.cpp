// A circuit given as a Python list of (gate name, q0, q1, theta) tuples, written
// as ccut_op rows.  Called through ctypes with the interpreter lock held; built
// into a library of its own, so that libccut.so needs no interpreter.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "ccut.h"

namespace {
// an int that fits 32 signed bits; nothing is raised
bool small_int(PyObject *o, int32_t &v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long x = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
  v = (int32_t)x;
  return true;
}
}  // namespace

// 0: out[0..n) written.  1: some op is not a 4-tuple of a name in `gates`, two
// ints of at most 32 bits and a float (or such an int): nothing is raised and
// the caller converts the ops itself.  n: the length `out` has room for.
extern "C" int ccut_pack_ops(PyObject *ops, PyObject *gates, Py_ssize_t n, ccut_op *out) {
  if (!PyList_CheckExact(ops) || !PyDict_CheckExact(gates) || PyList_GET_SIZE(ops) != n) return 1;
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject *t = PyList_GET_ITEM(ops, i);
    if (!PyTuple_CheckExact(t) || PyTuple_GET_SIZE(t) != 4) return 1;
    PyObject *name = PyTuple_GET_ITEM(t, 0), *th = PyTuple_GET_ITEM(t, 3);
    if (!PyUnicode_CheckExact(name)) return 1;
    PyObject *kind = PyDict_GetItemWithError(gates, name);
    int32_t k = 0, a = 0, b = 0, whole = 0;
    if (!kind) PyErr_Clear();
    if (!kind || !small_int(kind, k) || !small_int(PyTuple_GET_ITEM(t, 1), a) || !small_int(PyTuple_GET_ITEM(t, 2), b))
      return 1;
    double angle;
    if (PyFloat_CheckExact(th))
      angle = PyFloat_AS_DOUBLE(th);
    else if (small_int(th, whole))
      angle = whole;
    else
      return 1;
    out[i].kind = (uint32_t)k;
    out[i].q0 = (uint32_t)a;
    out[i].q1 = b >= 0 ? (uint32_t)b : 0;
    out[i].reserved = 0;
    out[i].theta = angle;
  }
  return 0;
}
