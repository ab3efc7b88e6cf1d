// Python module _call: the scan's two entry points of the C ABI called with torch tensors.
//
// A decode step is one kernel of some 4 us, and handing its sixteen arguments over through ctypes took
// 2.5 us of host time (on a slower host 6), beside a launch of 3.5.  Here the addresses are taken from the
// tensors directly and the options are put on the stack: 0.2 us (0.4).  The library is the one
// that ctypes has loaded; its entry points come in as addresses.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/m2rnn.h"

namespace {

decltype(&m2rnn_fwd_opt) fwd_opt = nullptr;
decltype(&m2rnn_bwd_opt) bwd_opt = nullptr;

// None -> NULL, an int as it is, a tensor -> its address, anything else -> what its data_ptr() says (a
// subclass of the tensor may have its own); false with a Python error set otherwise
bool address(PyObject *o, void *&p) {
  if (o == Py_None) {
    p = nullptr;
  } else if (THPVariable_CheckExact(o)) {
    p = THPVariable_Unpack(o).data_ptr();
  } else if (PyLong_Check(o)) {
    p = PyLong_AsVoidPtr(o);
    return !(p == nullptr && PyErr_Occurred());
  } else {
    PyObject *method = PyObject_GetAttrString(o, "data_ptr");
    if (!method) {
      if (PyErr_ExceptionMatches(PyExc_AttributeError))
        PyErr_SetString(PyExc_TypeError, "expected a tensor, an address or None");
      return false;
    }
    PyObject *number = PyObject_CallNoArgs(method);
    Py_DECREF(method);
    if (!number) return false;
    p = PyLong_AsVoidPtr(number);
    Py_DECREF(number);
    return !(p == nullptr && PyErr_Occurred());
  }
  return true;
}

// the addresses of the positional arguments a0 .. a0 + n - 1
template <size_t n>
bool addresses(PyObject *const *args, void *(&p)[n]) {
  try {
    for (size_t i = 0; i < n; ++i)
      if (!address(args[i], p[i])) return false;
  } catch (const std::exception &e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return false;
  }
  return true;
}

bool ready(const void *entry) {
  if (!entry) PyErr_SetString(PyExc_RuntimeError, "init has not been called");
  return entry != nullptr;
}

bool arity(Py_ssize_t have, Py_ssize_t want) {
  if (have != want) PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, have);
  return have == want;
}

PyObject *init(PyObject *, PyObject *const *args, Py_ssize_t n) {
  void *p[2];
  if (!arity(n, 2) || !addresses(args, p)) return nullptr;
  if (!p[0] || !p[1]) {
    PyErr_SetString(PyExc_ValueError, "an entry point is NULL");
    return nullptr;
  }
  fwd_opt = (decltype(fwd_opt))p[0];
  bwd_opt = (decltype(bwd_opt))p[1];
  Py_RETURN_NONE;
}

// fwd(desc, w_r, gate_alpha, gate_beta, q, k, v, f, W, H0, y, HT, ckpt, workspace, stream, bytes) -> status
PyObject *fwd(PyObject *, PyObject *const *args, Py_ssize_t n) {
  void *p[15];
  if (!ready((const void *)fwd_opt) || !arity(n, 16) || !addresses(args, p)) return nullptr;
  const size_t bytes = PyLong_AsSize_t(args[15]);
  if (bytes == (size_t)-1 && PyErr_Occurred()) return nullptr;
  m2rnn_opts o = {};
  o.w_r = p[1];
  o.gate_alpha = (const float *)p[2];
  o.gate_beta = (const float *)p[3];
  m2rnn_status st;
  Py_BEGIN_ALLOW_THREADS
  st = fwd_opt((const m2rnn_desc *)p[0], &o, p[4], p[5], p[6], (const float *)p[7], p[8], (const float *)p[9], p[10],
               (float *)p[11], (float *)p[12], p[13], bytes, p[14]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// bwd(desc, w_r, dw_r, gate_alpha, gate_beta, dgate_alpha, dgate_beta, q, k, v, f, W, H0, ckpt, dy, dHT,
//     dq, dk, dv, df, dW, dH0, workspace, stream, bytes, grad_clip) -> status
PyObject *bwd(PyObject *, PyObject *const *args, Py_ssize_t n) {
  void *p[24];
  if (!ready((const void *)bwd_opt) || !arity(n, 26) || !addresses(args, p)) return nullptr;
  const size_t bytes = PyLong_AsSize_t(args[24]);
  const double clip = PyFloat_AsDouble(args[25]);
  if (PyErr_Occurred()) return nullptr;
  m2rnn_opts o = {};
  o.w_r = p[1];
  o.dw_r = (float *)p[2];
  o.grad_clip = (float)clip;
  o.gate_alpha = (const float *)p[3];
  o.gate_beta = (const float *)p[4];
  o.dgate_alpha = (float *)p[5];
  o.dgate_beta = (float *)p[6];
  m2rnn_status st;
  Py_BEGIN_ALLOW_THREADS
  st = bwd_opt((const m2rnn_desc *)p[0], &o, p[7], p[8], p[9], (const float *)p[10], p[11], (const float *)p[12],
               (const float *)p[13], p[14], (const float *)p[15], p[16], p[17], p[18], (float *)p[19], (float *)p[20],
               (float *)p[21], p[22], bytes, p[23]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

PyMethodDef methods[] = {{"init", (PyCFunction)(void (*)(void))init, METH_FASTCALL, nullptr},
                         {"fwd", (PyCFunction)(void (*)(void))fwd, METH_FASTCALL, nullptr},
                         {"bwd", (PyCFunction)(void (*)(void))bwd, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__call() {
  PyObject *m = PyModule_Create(&module);
  // (a tensor is read through torch's own headers: under another torch its layout may be another one)
  if (m && PyModule_AddStringConstant(m, "torch_version", M2RNN_TORCH_VERSION) < 0) Py_CLEAR(m);
  return m;
}
