// binding.cpp -- the binding's small calls in native code.
//
// A call of a small product takes the GPU 2 to 5 us; its tensors' checks, output
// allocations and argument conversion took the Python interpreter 9 to 13.  Each
// function here does all of that for one entry point: it checks every tensor
// as the Python code does, allocates what the caller did not give, and calls
// the library.  It only takes calls in which everything is in order: for
// anything else (another type, device, layout, shape or size, a tensor
// subclass) it returns None before it does anything, and the Python code,
// which raises the errors, runs as it would without it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "mpc.h"

namespace {

struct Args {
  PyObject* const* a;
  int device;
  bool ok = true;

  // A plain tensor that is a contiguous int64 array on the device (n < 0: of
  // any size), or null with ok cleared.
  const at::Tensor* tensor(int i) {
    if (!THPVariable_CheckExact(a[i])) {
      ok = false;
      return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(a[i]);
    if (!t.defined() || t.scalar_type() != at::kLong || !t.device().is_cuda() || t.device().index() != device || !t.is_contiguous()) {
      ok = false;
      return nullptr;
    }
    return &t;
  }
  // Its data, if it has exactly n elements.
  uint64_t* exactly(int i, int64_t n) {
    const at::Tensor* t = ok ? tensor(i) : nullptr;
    if (!t || t->numel() != n) {
      ok = false;
      return nullptr;
    }
    return (uint64_t*)t->data_ptr();
  }
  uint64_t* at_least(int i, int64_t n) {
    const at::Tensor* t = ok ? tensor(i) : nullptr;
    if (!t || t->numel() < n) {
      ok = false;
      return nullptr;
    }
    return (uint64_t*)t->data_ptr();
  }
  uint64_t integer(int i) {
    const uint64_t v = PyLong_AsUnsignedLongLong(a[i]);
    if (PyErr_Occurred()) {  // not an integer, or out of range: the Python code says so
      PyErr_Clear();
      ok = false;
    }
    return v;
  }
  int small(int i) {
    const uint64_t v = integer(i);
    if (v > 1 << 20) ok = false;
    return (int)v;
  }
};

// Outputs: the caller's, or new tensors.
struct Out {
  at::Tensor made;
  PyObject* given = nullptr;
  uint64_t* ptr = nullptr;
  void take(Args& g, int i, int64_t n) {
    if (g.a[i] == Py_None) return;
    given = g.a[i];
    ptr = g.exactly(i, n);
  }
  void make(at::IntArrayRef shape, const at::Tensor& like) {
    if (given) return;
    made = at::empty(shape, like.options());
    ptr = (uint64_t*)made.data_ptr();
  }
  PyObject* object() {
    if (given) {
      Py_INCREF(given);
      return given;
    }
    return THPVariable_Wrap(std::move(made));
  }
};

// (status, z0, z1)
PyObject* result(int st, Out& z0, Out& z1) {
  PyObject *p0 = z0.object(), *p1 = z1.object();
  return Py_BuildValue("(iNN)", st, p0, p1);
}

#define FALL_BACK_UNLESS(cond) \
  if (!(cond)) Py_RETURN_NONE
mpc_ctx* context(PyObject* o) { return (mpc_ctx*)PyLong_AsVoidPtr(o); }

// share(ctx, device, x, src, tag, s0|None, s1|None)
PyObject* f_share(PyObject*, PyObject* const* a, Py_ssize_t n) {
  FALL_BACK_UNLESS(n == 7);
  HANDLE_TH_ERRORS
  Args g{a, (int)PyLong_AsLong(a[1])};
  const at::Tensor* x = g.tensor(2);
  const int src = g.small(3);
  const uint64_t tag = g.integer(4);
  FALL_BACK_UNLESS(g.ok);
  Out s0, s1;
  s0.take(g, 5, x->numel());
  s1.take(g, 6, x->numel());
  FALL_BACK_UNLESS(g.ok);
  s0.make(x->sizes(), *x);
  s1.make(x->sizes(), *x);
  mpc_status st;
  Py_BEGIN_ALLOW_THREADS st = mpc_share(context(a[0]), (const uint64_t*)x->data_ptr(), (size_t)x->numel(), src, tag, s0.ptr, s1.ptr);
  Py_END_ALLOW_THREADS return result(st, s0, s1);
  END_HANDLE_TH_ERRORS
}

// reveal(ctx, device, s0, s1, out|None) -> (status, out)
PyObject* f_reveal(PyObject*, PyObject* const* a, Py_ssize_t n) {
  FALL_BACK_UNLESS(n == 5);
  HANDLE_TH_ERRORS
  Args g{a, (int)PyLong_AsLong(a[1])};
  const at::Tensor* s0 = g.tensor(2);
  FALL_BACK_UNLESS(g.ok);
  const uint64_t* s1 = g.exactly(3, s0->numel());
  Out out;
  out.take(g, 4, s0->numel());
  FALL_BACK_UNLESS(g.ok);
  out.make(s0->sizes(), *s0);
  mpc_status st;
  Py_BEGIN_ALLOW_THREADS st = mpc_reveal(context(a[0]), (const uint64_t*)s0->data_ptr(), s1, (size_t)s0->numel(), out.ptr);
  Py_END_ALLOW_THREADS return Py_BuildValue("(iN)", st, out.object());
  END_HANDLE_TH_ERRORS
}

// beaver_mul(ctx, device, x0, x1, y0|None, y1|None, a0, a1, b0, b1, c0|None, c1|None, trunc, z0|None, z1|None)
PyObject* f_mul(PyObject*, PyObject* const* a, Py_ssize_t n) {
  FALL_BACK_UNLESS(n == 15);
  HANDLE_TH_ERRORS
  Args g{a, (int)PyLong_AsLong(a[1])};
  const at::Tensor* x0 = g.tensor(2);
  FALL_BACK_UNLESS(g.ok);
  const int64_t len = x0->numel();
  const uint64_t* x1 = g.exactly(3, len);
  const bool square = a[4] == Py_None && a[5] == Py_None;
  const uint64_t *y0 = square ? nullptr : g.exactly(4, len), *y1 = square ? nullptr : g.exactly(5, len);
  mpc_triple t{g.at_least(6, len), g.at_least(7, len), g.at_least(8, len), g.at_least(9, len), nullptr, nullptr};
  // (a square ignores c, and takes a triple that has one)
  if (!square || a[10] != Py_None) t.c0 = square ? g.at_least(10, 0) : g.at_least(10, len);
  if (!square || a[11] != Py_None) t.c1 = square ? g.at_least(11, 0) : g.at_least(11, len);
  const int trunc = g.small(12);
  Out z0, z1;
  z0.take(g, 13, len);
  z1.take(g, 14, len);
  FALL_BACK_UNLESS(g.ok);
  z0.make(x0->sizes(), *x0);
  z1.make(x0->sizes(), *x0);
  mpc_status st;
  Py_BEGIN_ALLOW_THREADS st = mpc_beaver_mul(context(a[0]), (size_t)len, (const uint64_t*)x0->data_ptr(), x1, y0, y1, &t, trunc, z0.ptr, z1.ptr);
  Py_END_ALLOW_THREADS return result(st, z0, z1);
  END_HANDLE_TH_ERRORS
}

// beaver_matmul(ctx, device, x0, x1, y0, y1, a0, a1, b0, b1, c0, c1, trunc, form, z0|None, z1|None)
PyObject* f_matmul(PyObject*, PyObject* const* a, Py_ssize_t n) {
  FALL_BACK_UNLESS(n == 16);
  HANDLE_TH_ERRORS
  Args g{a, (int)PyLong_AsLong(a[1])};
  const at::Tensor *x0 = g.tensor(2), *y0 = g.tensor(4);
  FALL_BACK_UNLESS(g.ok && x0->dim() == 2 && y0->dim() == 2 && x0->size(1) == y0->size(0));
  const int64_t M = x0->size(0), K = x0->size(1), N = y0->size(1);
  const uint64_t *x1 = g.exactly(3, M * K), *y1 = g.exactly(5, K * N);
  const mpc_triple t{g.at_least(6, M * K), g.at_least(7, M * K), g.at_least(8, K * N), g.at_least(9, K * N), g.at_least(10, M * N), g.at_least(11, M * N)};
  const int trunc = g.small(12), form = g.small(13);
  Out z0, z1;
  z0.take(g, 14, M * N);
  z1.take(g, 15, M * N);
  FALL_BACK_UNLESS(g.ok);
  z0.make({M, N}, *x0);
  z1.make({M, N}, *x0);
  mpc_status st;
  Py_BEGIN_ALLOW_THREADS st = mpc_beaver_matmul(context(a[0]), M, N, K, (const uint64_t*)x0->data_ptr(), x1, (const uint64_t*)y0->data_ptr(), y1, &t,
                                                trunc, (mpc_form)form, z0.ptr, z1.ptr);
  Py_END_ALLOW_THREADS return result(st, z0, z1);
  END_HANDLE_TH_ERRORS
}

#define FAST(name, f) {name, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST("share", f_share), FAST("reveal", f_reveal), FAST("beaver_mul", f_mul), FAST("beaver_matmul", f_matmul),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
