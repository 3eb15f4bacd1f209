// The two calls a program makes per linear and token, dpllm_gemv and dpllm_estimate, for Python: what binding.py does through
// ctypes, without a Python object per argument.  us of host time per call of a loop, ctypes -> here: dpllm_gemv 4.3 -> 3.4, of which the
// launch is 2.5.
// A call that is out of the ordinary in any way (an argument that is no int or has no data_ptr(), a closed model) is not made here:
// the answer is kElsewhere and binding.py makes it the long way, with the errors that has.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

namespace {

constexpr long kElsewhere = 1;

using Gemv = int (*)(void*, int, int, const int32_t*, const void*, void*, int, void*);
using Estimate = int (*)(void*, int, int, int, const void*, float*, int32_t*, void*);
Gemv the_gemv = nullptr;
Estimate the_estimate = nullptr;
PyObject *get_device = nullptr, *get_stream = nullptr;   // torch._C._cuda_getDevice, _cuda_getCurrentRawStream
PyObject *s_data_ptr = nullptr, *s_dim = nullptr, *s_size = nullptr, *zero = nullptr;

// A C int as ctypes converts one; false: no int.
bool as_int(PyObject* o, int* v) {
  if (!PyLong_Check(o)) return false;
  *v = (int)PyLong_AsUnsignedLongMask(o);
  return true;
}

// false: not to be had (no error is left behind)
bool address(PyObject* o, void** p) {
  PyObject* a = PyLong_Check(o) ? Py_NewRef(o) : PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (a != nullptr && PyLong_Check(a)) {
    *p = PyLong_AsVoidPtr(a);
    Py_DECREF(a);
    if (!PyErr_Occurred()) return true;
  } else {
    Py_XDECREF(a);
  }
  PyErr_Clear();
  return false;
}

bool tensor(PyObject* o, void** p) { return !PyLong_Check(o) && address(o, p); }

// the current stream of the current device
bool stream(void** p) {
  PyObject* d = PyObject_CallNoArgs(get_device);
  PyObject* s = d != nullptr ? PyObject_CallOneArg(get_stream, d) : nullptr;
  const bool ok = s != nullptr && PyLong_Check(s);
  if (ok) *p = PyLong_AsVoidPtr(s);
  Py_XDECREF(d);
  Py_XDECREF(s);
  if (!ok || PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

// samples of x: 1 for a vector, else its first dimension
bool samples(PyObject* x, int* n) {
  PyObject* d = PyObject_CallMethodNoArgs(x, s_dim);
  int dim = 0;
  bool ok = d != nullptr && as_int(d, &dim);
  Py_XDECREF(d);
  *n = 1;
  if (ok && dim != 1) {
    PyObject* s = PyObject_CallMethodOneArg(x, s_size, zero);
    ok = s != nullptr && as_int(s, n);
    Py_XDECREF(s);
  }
  if (!ok) PyErr_Clear();
  return ok;
}

// bind(address of dpllm_gemv, of dpllm_estimate, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *g = nullptr, *e = nullptr;
  if (n != 4 || !address(a[0], &g) || !address(a[1], &e)) {
    PyErr_SetString(PyExc_TypeError, "bind(gemv, estimate, get_device, get_stream)");
    return nullptr;
  }
  the_gemv = reinterpret_cast<Gemv>(g);
  the_estimate = reinterpret_cast<Estimate>(e);
  Py_XSETREF(get_device, Py_NewRef(a[2]));
  Py_XSETREF(get_stream, Py_NewRef(a[3]));
  Py_RETURN_NONE;
}

// gemv(model, id, k, x, y, k_dev or None)
PyObject* gemv(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *m = nullptr, *x = nullptr, *y = nullptr, *kd = nullptr, *st = nullptr;
  int id = 0, k = 0, b = 0;
  if (n != 6 || the_gemv == nullptr || !PyLong_Check(a[0]) || !address(a[0], &m) || m == nullptr || !as_int(a[1], &id) || !as_int(a[2], &k) ||
      !tensor(a[3], &x) || !tensor(a[4], &y) || (a[5] != Py_None && !tensor(a[5], &kd)) || !samples(a[3], &b) || !stream(&st))
    return PyLong_FromLong(kElsewhere);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = the_gemv(m, id, k, static_cast<const int32_t*>(kd), x, y, b, st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// estimate(model, id, l, h, x, e_out, k_out)
PyObject* estimate(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *m = nullptr, *x = nullptr, *e = nullptr, *ko = nullptr, *st = nullptr;
  int id = 0, l = 0, h = 0;
  if (n != 7 || the_estimate == nullptr || !PyLong_Check(a[0]) || !address(a[0], &m) || m == nullptr || !as_int(a[1], &id) || !as_int(a[2], &l) ||
      !as_int(a[3], &h) || !tensor(a[4], &x) || !tensor(a[5], &e) || !tensor(a[6], &ko) || !stream(&st))
    return PyLong_FromLong(kElsewhere);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = the_estimate(m, id, l, h, x, static_cast<float*>(e), static_cast<int32_t*>(ko), st);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

using Fast = PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t);
PyCFunction as_method(Fast f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }
PyMethodDef methods[] = {{"bind", as_method(bind), METH_FASTCALL, nullptr},
                         {"gemv", as_method(gemv), METH_FASTCALL, nullptr},
                         {"estimate", as_method(estimate), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef definition = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_dim = PyUnicode_InternFromString("dim");
  s_size = PyUnicode_InternFromString("size");
  zero = PyLong_FromLong(0);
  if (s_data_ptr == nullptr || s_dim == nullptr || s_size == nullptr || zero == nullptr) return nullptr;
  PyObject* m = PyModule_Create(&definition);
  if (m != nullptr && PyModule_AddIntConstant(m, "ELSEWHERE", kElsewhere) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
