// The way from Python to the entry points that a layer's pass goes through (binding.py), for calls whose arguments are what they
// should be: plain tensors and plain ints.  Each function here reads the tensors' pointers, sizes and types, calls
// the C entry point on the current stream and returns its code; for anything else it returns None and has done nothing, and
// binding.py takes the general way, through ctypes, which also names the error.  What is checked is what the general way checks: that
// a quantiser's input lies in device memory with rows of unit stride, and the types of inputs and Y.  Every other tensor is a pointer.
//
// Why: a call through ctypes costs the host 1.7 us (a quantiser, 10 arguments) to 2.3 us (a layer, 19) before the launch, against
// 3.4 us of the runtime's own, and a decode pass of two calls was bound by that.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>

#include "../../include/serq.h"

namespace {

decltype(&serq_quantize_act) f_quantize_act;
decltype(&serq_swiglu_quantize_act) f_swiglu_quantize_act;
decltype(&serq_mx_quantize_act) f_mx_quantize_act;
decltype(&serq_mx_swiglu_quantize_act) f_mx_swiglu_quantize_act;
decltype(&serq_quantize_act_asym) f_quantize_act_asym;
decltype(&serq_linear) f_linear;
decltype(&serq_mx_linear) f_mx_linear;
decltype(&serq_g128_linear) f_g128_linear;

// Arguments of one call; `ok` falls once one of them is not the plain thing.
struct Args {
  PyObject* const* a;
  bool ok = !at::impl::torch_function_mode_enabled();

  const at::Tensor* tensor(int i) {                    // a plain tensor or parameter, of any type and any number of dimensions
    if (!THPVariable_CheckExact(a[i])) { ok = false; return nullptr; }
    return &THPVariable_Unpack(a[i]);
  }
  void* ptr(int i) {                                   // of a tensor
    const at::Tensor* t = ok ? tensor(i) : nullptr;
    return t ? t->data_ptr() : nullptr;
  }
  void* ptr_or_none(int i) { return a[i] == Py_None ? nullptr : ptr(i); }
  int64_t integer(int i) {
    int over = 1;
    long long v = 0;
    if (PyLong_CheckExact(a[i])) v = PyLong_AsLongLongAndOverflow(a[i], &over);
    if (over) ok = false;
    return v;
  }
  int integer32(int i) {
    const int64_t v = integer(i);
    if (v != (int)v) ok = false;
    return (int)v;
  }
  int dtype(const at::Tensor& t) {
    switch (t.scalar_type()) {
      case at::kFloat: return SERQ_F32;
      case at::kHalf: return SERQ_F16;
      case at::kBFloat16: return SERQ_BF16;
      default: ok = false; return 0;
    }
  }
  // [M, K] activations with unit inner stride
  struct Rows { void* p; int dt; int64_t M, K, ld; };
  Rows rows(int i) {
    Rows r{};
    const at::Tensor* t = ok ? tensor(i) : nullptr;
    if (!t || !t->is_cuda() || t->dim() != 2 || t->stride(1) != 1) { ok = false; return r; }
    r = {t->data_ptr(), dtype(*t), t->size(0), t->size(1), 0};
    r.ld = r.M > 0 ? t->stride(0) : r.K;
    return r;
  }
  // the two halves of a gated product, alike in shape and type
  void alike(const Rows& g, const Rows& u) {
    if (g.M != u.M || g.K != u.K || g.dt != u.dt) ok = false;
  }
};

void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// n arguments in; `read` takes them and returns the call, which is made if everything was plain.
// The interpreter lock is given up for the call proper, as ctypes does: a launch waits where the queue is full, and what it waits for
// may be a host function that needs the lock.  The caller's frame holds the arguments meanwhile.  (Host time of a decode pass of two
// calls, lock held / given up: 7.9 / 8.0 us.)
template <class F>
PyObject* run(PyObject* const* a, Py_ssize_t n, Py_ssize_t want, const F& read) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected", want);
    return nullptr;
  }
  int rc = 0;
  PyThreadState* unlocked = nullptr;
  try {
    Args x{a};
    const auto call = read(x);
    if (!x.ok) Py_RETURN_NONE;
    void* const st = stream();
    unlocked = PyEval_SaveThread();
    rc = call(st);
  } catch (...) {                                      // (a tensor without storage, for instance: the general way says which)
    if (unlocked) PyEval_RestoreThread(unlocked);
    Py_RETURN_NONE;
  }
  PyEval_RestoreThread(unlocked);
  return PyLong_FromLong(rc);
}

PyObject* quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n) {        // X, s_inv, abits, Xq, scale
  return run(a, n, 5, [](Args& x) {
    const Args::Rows X = x.rows(0);
    const float* s = (const float*)x.ptr_or_none(1);
    const int abits = x.integer32(2);
    void* xq = x.ptr(3);
    float* sc = (float*)x.ptr(4);
    return [=](void* st) { return f_quantize_act(X.p, X.dt, s, X.M, X.K, X.ld, abits, xq, sc, st); };
  });
}

PyObject* swiglu_quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n) {  // G, U, s_inv, abits, Xq, scale
  return run(a, n, 6, [](Args& x) {
    const Args::Rows G = x.rows(0), U = x.rows(1);
    const float* s = (const float*)x.ptr_or_none(2);
    const int abits = x.integer32(3);
    void* xq = x.ptr(4);
    float* sc = (float*)x.ptr(5);
    x.alike(G, U);
    return [=](void* st) { return f_swiglu_quantize_act(G.p, U.p, G.dt, s, G.M, G.K, G.ld, U.ld, abits, xq, sc, st); };
  });
}

PyObject* mx_quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n) {     // X, s_inv, Xq, xsc
  return run(a, n, 4, [](Args& x) {
    const Args::Rows X = x.rows(0);
    const float* s = (const float*)x.ptr_or_none(1);
    void* xq = x.ptr(2);
    uint8_t* sc = (uint8_t*)x.ptr(3);
    return [=](void* st) { return f_mx_quantize_act(X.p, X.dt, s, X.M, X.K, X.ld, xq, sc, st); };
  });
}

PyObject* mx_swiglu_quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n) {   // G, U, s_inv, Xq, xsc
  return run(a, n, 5, [](Args& x) {
    const Args::Rows G = x.rows(0), U = x.rows(1);
    const float* s = (const float*)x.ptr_or_none(2);
    void* xq = x.ptr(3);
    uint8_t* sc = (uint8_t*)x.ptr(4);
    x.alike(G, U);
    return [=](void* st) { return f_mx_swiglu_quantize_act(G.p, U.p, G.dt, s, G.M, G.K, G.ld, U.ld, xq, sc, st); };
  });
}

PyObject* quantize_act_asym(PyObject*, PyObject* const* a, Py_ssize_t n) {   // X, s_inv, abits, Xq, scale, zero
  return run(a, n, 6, [](Args& x) {
    const Args::Rows X = x.rows(0);
    const float* s = (const float*)x.ptr_or_none(1);
    const int abits = x.integer32(2);
    void* xq = x.ptr(3);
    float* sc = (float*)x.ptr(4);
    int32_t* z = (int32_t*)x.ptr(5);
    return [=](void* st) { return f_quantize_act_asym(X.p, X.dt, s, X.M, X.K, X.ld, abits, xq, sc, z, st); };
  });
}

// Y: a tensor of a type the library has, and its row stride
struct Out { void* p; int dt; int64_t ld; };
Out output(Args& x, int i) {
  Out y{};
  const at::Tensor* t = x.ok ? x.tensor(i) : nullptr;
  if (!t || t->dim() < 1) { x.ok = false; return y; }
  y = {t->data_ptr(), x.dtype(*t), t->stride(0)};
  return y;
}
struct Room { void* p; size_t n; };
Room workspace(Args& x, int i) {
  Room r{};
  if (x.a[i] == Py_None) return r;
  const at::Tensor* t = x.ok ? x.tensor(i) : nullptr;
  if (t) r = {t->data_ptr(), (size_t)t->numel()};
  return r;
}

// Xq, scale, abits, Wq, wscale, s_begin, r, Rp, r_dtype, M, N, K, Y, ws, flags
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return run(a, n, 15, [](Args& x) {
    const void* xq = x.ptr(0);
    const float* sc = (const float*)x.ptr(1);
    const int abits = x.integer32(2);
    const void* wq = x.ptr(3);
    const float* wsc = (const float*)x.ptr(4);
    const int s0 = x.integer32(5), r = x.integer32(6);
    const void* rp = x.ptr_or_none(7);
    const int rdt = x.integer32(8);
    const int64_t M = x.integer(9), N = x.integer(10), K = x.integer(11);
    const Out y = output(x, 12);
    const Room w = workspace(x, 13);
    const int flags = x.integer32(14);
    return [=](void* st) { return f_linear(xq, sc, abits, wq, wsc, s0, r, rp, rdt, M, N, K, y.p, y.dt, y.ld, w.p, w.n, flags, st); };
  });
}

// Xq, xsc, Wq, wsc, s_begin, r, Rq, rsc, M, N, K, Y, ws, flags
PyObject* mx_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return run(a, n, 14, [](Args& x) {
    const void* xq = x.ptr(0);
    const uint8_t* xsc = (const uint8_t*)x.ptr(1);
    const void* wq = x.ptr(2);
    const uint8_t* wsc = (const uint8_t*)x.ptr(3);
    const int s0 = x.integer32(4), r = x.integer32(5);
    const void* rq = x.ptr_or_none(6);
    const uint8_t* rsc = (const uint8_t*)x.ptr_or_none(7);
    const int64_t M = x.integer(8), N = x.integer(9), K = x.integer(10);
    const Out y = output(x, 11);
    const Room w = workspace(x, 12);
    const int flags = x.integer32(13);
    return [=](void* st) { return f_mx_linear(xq, xsc, wq, wsc, s0, r, rq, rsc, M, N, K, y.p, y.dt, M > 0 ? y.ld : N, w.p, w.n, flags, st); };
  });
}

// Xq, scale, zero, abits, Wq, gscale, wsum, s_begin, r, Rp, r_dtype, M, N, K, Y, flags
PyObject* g128_linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return run(a, n, 16, [](Args& x) {
    const void* xq = x.ptr(0);
    const float* sc = (const float*)x.ptr(1);
    const int32_t* z = (const int32_t*)x.ptr_or_none(2);
    const int abits = x.integer32(3);
    const void *wq = x.ptr(4), *gsc = x.ptr(5);
    const float* wsum = (const float*)x.ptr(6);
    const int s0 = x.integer32(7), r = x.integer32(8);
    const void* rp = x.ptr_or_none(9);
    const int rdt = x.integer32(10);
    const int64_t M = x.integer(11), N = x.integer(12), K = x.integer(13);
    const Out y = output(x, 14);
    const int flags = x.integer32(15);
    return [=](void* st) { return f_g128_linear(xq, sc, z, abits, wq, gsc, wsum, s0, r, rp, rdt, M, N, K, y.p, y.dt, y.ld, flags, st); };
  });
}

// the addresses of the entry points, in the order of the declarations above
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void** const slots[] = {(void**)&f_quantize_act, (void**)&f_swiglu_quantize_act, (void**)&f_mx_quantize_act,
                          (void**)&f_mx_swiglu_quantize_act, (void**)&f_quantize_act_asym, (void**)&f_linear,
                          (void**)&f_mx_linear, (void**)&f_g128_linear};
  if (n != (Py_ssize_t)(sizeof(slots) / sizeof(slots[0]))) {
    PyErr_SetString(PyExc_TypeError, "one address per entry point expected");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    void* p = PyLong_AsVoidPtr(a[i]);
    if (!p) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
    *slots[i] = p;
  }
  Py_RETURN_NONE;
}

#define SERQ_FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SERQ_FAST(bind), SERQ_FAST(quantize_act), SERQ_FAST(swiglu_quantize_act), SERQ_FAST(mx_quantize_act),
                         SERQ_FAST(mx_swiglu_quantize_act), SERQ_FAST(quantize_act_asym), SERQ_FAST(linear),
                         SERQ_FAST(mx_linear), SERQ_FAST(g128_linear), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
