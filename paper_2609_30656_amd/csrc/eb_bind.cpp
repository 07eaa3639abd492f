// _ebbind — the argument marshalling of the library's hot entry points as a
// CPython extension: torch tensors in, one call of the C ABI out.
//
// A call through ctypes spends 1.5 us on each tensor's checks and descriptor
// and 1 us on the foreign call, 6 us in all where the smallest lookup's kernel
// takes 3 (64 bags of one table, called back to back: 6.2 us a call through
// ctypes, 4.0 through this; 26 tables, 50 examples with the FM term 10.5 and
// 7.1).  Only the plain case is handled: each
// argument is None or an exact torch.Tensor (or Parameter) that passes the
// checks.  For anything else a function returns NotImplemented and the caller
// takes the ctypes path, which makes the same checks and raises their errors.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include "eb.h"

namespace {

decltype(&eb_forward) p_forward;
decltype(&eb_forward_seq) p_forward_seq;
decltype(&eb_fm_cross) p_fm_cross;
decltype(&eb_forward_fm) p_forward_fm;
decltype(&eb_backward_update) p_backward;
decltype(&eb_backward_update_noalloc) p_backward_noalloc;

// The eb_tensor of o on GPU `device`; false if o is not the plain case.
bool describe(PyObject *o, long device, eb_tensor *t) {
  if (o == Py_None) {
    *t = {nullptr, 0, EB_T_F32};
    return true;
  }
  if (!THPVariable_CheckExact(o)) return false;
  try {
    const at::Tensor &x = THPVariable_Unpack(o);
    if (!x.is_cuda() || x.get_device() != device || x.layout() != at::kStrided || !x.is_contiguous()) return false;
    t->numel = x.numel();
    t->data = t->numel ? x.data_ptr() : nullptr;
    switch (x.scalar_type()) {
      case at::kInt: t->elem_type = EB_I32; break;
      case at::kLong: t->elem_type = EB_I64; break;
      case at::kFloat: t->elem_type = EB_T_F32; break;
      default: return false;
    }
    return true;
  } catch (...) {
    return false;  // no storage, a wrapped tensor, ...
  }
}

// Arguments of one call: (handle or None, device, tensors and scalars ...).
struct Args {
  PyObject *const *v;
  Py_ssize_t n;
  const eb_tables *handle = nullptr;
  long device = -1;
  bool plain = true;

  Args(PyObject *const *args, Py_ssize_t nargs, Py_ssize_t want) : v(args), n(nargs) {
    if (n != want) {
      PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
      plain = false;
      return;
    }
    if (v[0] != Py_None) handle = static_cast<const eb_tables *>(PyLong_AsVoidPtr(v[0]));
    device = PyLong_AsLong(v[1]);
    plain = !PyErr_Occurred() && !at::impl::torch_function_mode_enabled();
  }
  eb_tensor tensor(int i) {
    eb_tensor t = {nullptr, 0, EB_T_F32};
    plain = plain && describe(v[i], device, &t);
    return t;
  }
  long integer(int i) {
    const long x = plain ? PyLong_AsLong(v[i]) : 0;
    plain = plain && !PyErr_Occurred();
    return x;
  }
  double real(int i) {
    const double x = plain ? PyFloat_AsDouble(v[i]) : 0.0;
    plain = plain && !PyErr_Occurred();
    return x;
  }
};

template <typename F>
PyObject *finish(const Args &a, F call) {
  if (PyErr_Occurred()) return nullptr;
  if (!a.plain) Py_RETURN_NOTIMPLEMENTED;
  eb_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

PyObject *forward(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Args a(args, n, 7);
  if (n != 7) return nullptr;
  const eb_tensor i = a.tensor(2), o = a.tensor(3), w = a.tensor(4), out = a.tensor(6);
  const long mode = a.integer(5);
  return finish(a, [&] { return p_forward(a.handle, i, o, w, static_cast<eb_pooling>(mode), out); });
}

PyObject *forward_seq(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Args a(args, n, 5);
  if (n != 5) return nullptr;
  const eb_tensor i = a.tensor(2), o = a.tensor(3), out = a.tensor(4);
  return finish(a, [&] { return p_forward_seq(a.handle, i, o, out); });
}

PyObject *fm_cross(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Args a(args, n, 4);
  if (n != 4) return nullptr;
  const eb_tensor p = a.tensor(2), f = a.tensor(3);
  return finish(a, [&] { return p_fm_cross(a.handle, p, f); });
}

PyObject *forward_fm(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Args a(args, n, 8);
  if (n != 8) return nullptr;
  const eb_tensor i = a.tensor(2), o = a.tensor(3), w = a.tensor(4), out = a.tensor(6), f = a.tensor(7);
  const long mode = a.integer(5);
  return finish(a, [&] { return p_forward_fm(a.handle, i, o, w, static_cast<eb_pooling>(mode), out, f); });
}

// ..., optimizer, learning rate, eps, state, and for backward_update the
// workspace's address and bytes
PyObject *backward(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Args a(args, n, 13);
  if (n != 13) return nullptr;
  const eb_tensor i = a.tensor(2), o = a.tensor(3), w = a.tensor(4), g = a.tensor(6), s = a.tensor(10);
  const long mode = a.integer(5), opt = a.integer(7), bytes = a.integer(12);
  const float lr = static_cast<float>(a.real(8)), eps = static_cast<float>(a.real(9));
  void *ws = a.plain ? PyLong_AsVoidPtr(a.v[11]) : nullptr;
  return finish(a, [&] {
    return p_backward(a.handle, i, o, w, static_cast<eb_pooling>(mode), g, static_cast<int32_t>(opt), lr, eps, s, ws,
                      static_cast<size_t>(bytes));
  });
}

PyObject *backward_noalloc(PyObject *, PyObject *const *args, Py_ssize_t n) {
  Args a(args, n, 11);
  if (n != 11) return nullptr;
  const eb_tensor i = a.tensor(2), o = a.tensor(3), w = a.tensor(4), g = a.tensor(6), s = a.tensor(10);
  const long mode = a.integer(5), opt = a.integer(7);
  const float lr = static_cast<float>(a.real(8)), eps = static_cast<float>(a.real(9));
  return finish(a, [&] {
    return p_backward_noalloc(a.handle, i, o, w, static_cast<eb_pooling>(mode), g, static_cast<int32_t>(opt), lr, eps, s);
  });
}

// bind(address of eb_forward, eb_forward_seq, eb_fm_cross, eb_forward_fm,
// eb_backward_update, eb_backward_update_noalloc): the loaded library's.
PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 6) {
    PyErr_SetString(PyExc_TypeError, "bind takes six addresses");
    return nullptr;
  }
  void *p[6];
  for (int k = 0; k < 6; ++k) p[k] = PyLong_AsVoidPtr(args[k]);
  if (PyErr_Occurred()) return nullptr;
  p_forward = reinterpret_cast<decltype(p_forward)>(p[0]);
  p_forward_seq = reinterpret_cast<decltype(p_forward_seq)>(p[1]);
  p_fm_cross = reinterpret_cast<decltype(p_fm_cross)>(p[2]);
  p_forward_fm = reinterpret_cast<decltype(p_forward_fm)>(p[3]);
  p_backward = reinterpret_cast<decltype(p_backward)>(p[4]);
  p_backward_noalloc = reinterpret_cast<decltype(p_backward_noalloc)>(p[5]);
  Py_RETURN_NONE;
}

#define EB_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {EB_METHOD(bind),       EB_METHOD(forward),  EB_METHOD(forward_seq),      EB_METHOD(fm_cross),
                         EB_METHOD(forward_fm), EB_METHOD(backward), EB_METHOD(backward_noalloc), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ebbind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ebbind(void) { return PyModule_Create(&module); }
