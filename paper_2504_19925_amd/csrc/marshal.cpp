// Argument marshalling of the device calls, in C++: the checks of binding.py (exact tensor type, on
// the GPU, dtype, contiguous, size) and the call itself, about half a microsecond per call where
// ctypes and attribute look-ups take five to fifteen.  A small layer's iteration is a dozen calls
// whose kernels run a few microseconds each, so the host sets its pace (8 experts of 128 x 256,
// 1024 tokens, fp32: 221 us of host time per step, 125 us of kernels).
//
// Every function takes the positional arguments of its namesake in binding.py and returns the
// library's status, or None when an argument is not of the plain form (a keyword, a tensor subclass,
// a wrong dtype, too few elements, ...): binding.py then goes through its own checks, which accept it
// or raise the error that names it.  Nothing is kept between calls.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <utility>

#include "symi.h"

namespace {

#define SYMI_CALLS(X)                                                                          \
  X(symi_route) X(symi_route_bwd) X(symi_place) X(symi_dispatch) X(symi_dispatch_noalloc)      \
  X(symi_dispatch_capacity) X(symi_dispatch_bwd) X(symi_expert_fwd) X(symi_expert_bwd)         \
  X(symi_expert_bwd_slots) X(symi_expert_bwd_active) X(symi_replica_allreduce)                 \
  X(symi_router_fwd) X(symi_router_bwd) X(symi_combine) X(symi_combine_bwd)                    \
  X(symi_adam_to_replicas) X(symi_adam_to_replicas_active) X(symi_workspace_bytes)

// entry points of the loaded libsymi.so (addresses handed over by attach)
struct Entries {
#define X(name) decltype(&::name) name = nullptr;
  SYMI_CALLS(X)
#undef X
} g;
PyTypeObject* g_ctx_type = nullptr;    // binding.SymiCtx
PyTypeObject* g_adam_type = nullptr;   // binding.SymiAdam
PyObject *g_ptr = nullptr, *g_cfg = nullptr;   // interned attribute names

// one argument of a C call: converts to the type of the parameter it is passed for
struct Val {
  void* p = nullptr;
  int i = 0;
  float f = 0.f;
  template <class T> operator T*() const { return static_cast<T*>(p); }
  operator int() const { return i; }
  operator float() const { return f; }
};

// the bytes of a ctypes object, copied out
template <class T>
bool read_ctypes(PyObject* o, T& out) {
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return false;
  }
  const bool ok = b.len == (Py_ssize_t)sizeof(T);
  if (ok) memcpy(&out, b.buf, sizeof(T));
  PyBuffer_Release(&b);
  return ok;
}

class Call {
 public:
  symi_cfg c;
  long long T, E, S, A, d, f, nw, ne;
  bool ok = false;

  Call(PyObject* const* a, Py_ssize_t n, Py_ssize_t expected) : a_(a) {
    if (n != expected || !g.symi_workspace_bytes || Py_TYPE(a[0]) != g_ctx_type) return;
    PyObject* p = PyObject_GetAttr(a[0], g_ptr);
    PyObject* q = PyObject_GetAttr(a[0], g_cfg);
    ok = p && q && p != Py_None && read_ctypes(p, ctx_) && read_ctypes(q, c) && ctx_;
    Py_XDECREF(p);
    Py_XDECREF(q);
    if (!ok) {
      PyErr_Clear();
      return;
    }
    T = c.T; E = c.E; S = c.S_tot; d = c.d; f = c.f;
    A = (long long)c.T * c.k;
    nw = S * d * f;
    ne = E * d * f;
  }
  Val act(int i, long long n) { return tensor(i, c.dtype == SYMI_BF16 ? at::kBFloat16 : at::kFloat, n); }
  Val f32(int i, long long n) { return tensor(i, at::kFloat, n); }
  Val i32(int i, long long n) { return tensor(i, at::kInt, n); }
  Val ws(int i) { return ok ? tensor(i, at::kByte, (long long)g.symi_workspace_bytes(&c)) : Val(); }
  Val f32_or_none(int i, long long n) { return a_[i] == Py_None ? Val() : f32(i, n); }
  Val integer(int i) {
    Val v;
    if (!PyLong_CheckExact(a_[i])) { ok = false; return v; }
    const long x = PyLong_AsLong(a_[i]);
    if ((x == -1 && PyErr_Occurred()) || x != (int)x) { PyErr_Clear(); ok = false; return v; }
    v.i = (int)x;
    return v;
  }
  Val real(int i) {
    Val v;
    if (!PyFloat_CheckExact(a_[i])) { ok = false; return v; }
    v.f = (float)PyFloat_AS_DOUBLE(a_[i]);
    return v;
  }
  Val adam(int i) {
    Val v;
    if (Py_TYPE(a_[i]) != g_adam_type || !read_ctypes(a_[i], hp_)) { ok = false; return v; }
    v.p = &hp_;
    return v;
  }
  template <class Fn, size_t N>
  PyObject* operator()(Fn fn, const Val (&v)[N]) {
    if (!ok || !fn) Py_RETURN_NONE;
    return run(fn, v, std::make_index_sequence<N>());
  }

 private:
  Val tensor(int i, at::ScalarType type, long long n) {
    Val v;
    if (!ok) return v;
    ok = false;
    if (!THPVariable_CheckExact(a_[i])) return v;
    try {
      const at::Tensor& t = THPVariable_Unpack(a_[i]);
      if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || !t.is_contiguous() || t.numel() < n) return v;
      v.p = t.data_ptr();
      ok = true;
    } catch (...) {   // a tensor without storage: the slow path says so
    }
    return v;
  }
  template <class Fn, size_t N, size_t... I>
  PyObject* run(Fn fn, const Val (&v)[N], std::index_sequence<I...>) {
    int rc = 0;
    try {
      void* const stream = c10::hip::getCurrentHIPStream().stream();
      Py_BEGIN_ALLOW_THREADS
      rc = fn(ctx_, v[I]..., stream);
      Py_END_ALLOW_THREADS
    } catch (const std::exception& e) {
      PyErr_SetString(PyExc_RuntimeError, e.what());
      return nullptr;
    }
    return PyLong_FromLong(rc);
  }
  PyObject* const* a_;
  symi_ctx* ctx_ = nullptr;
  symi_adam hp_;
};

#define DEF(name) PyObject* py_##name(PyObject*, PyObject* const* a, Py_ssize_t n)

DEF(symi_route) {
  Call c(a, n, 5);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.f32(1, c.T * c.E), c.i32(2, c.A), c.f32(3, c.A), c.i32(4, c.E)};
  return c(g.symi_route, v);
}
DEF(symi_route_bwd) {
  Call c(a, n, 6);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.f32(1, c.T * c.E), c.i32(2, c.A), c.f32(3, c.A), c.f32(4, c.A), c.f32(5, c.T * c.E)};
  return c(g.symi_route_bwd, v);
}
DEF(symi_place) {
  Call c(a, n, 5);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.i32(1, c.E), c.i32(2, c.E), c.i32(3, c.S), c.i32(4, c.E + 1)};
  return c(g.symi_place, v);
}
DEF(symi_dispatch) {
  Call c(a, n, 11);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.T * c.d), c.i32(2, c.A), c.i32(3, c.E), c.i32(4, c.E), c.i32(5, c.E + 1), c.i32(6, c.A),
                   c.i32(7, c.A), c.i32(8, c.S + 1), c.act(9, c.A * c.d), c.ws(10)};
  return c(g.symi_dispatch, v);
}
DEF(symi_dispatch_noalloc) {
  Call c(a, n, 10);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.T * c.d), c.i32(2, c.A), c.i32(3, c.E), c.i32(4, c.E), c.i32(5, c.E + 1), c.i32(6, c.A),
                   c.i32(7, c.A), c.i32(8, c.S + 1), c.act(9, c.A * c.d)};
  return c(g.symi_dispatch_noalloc, v);
}
DEF(symi_dispatch_capacity) {
  Call c(a, n, 12);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.integer(1), c.act(2, c.T * c.d), c.i32(3, c.A), c.i32(4, c.E), c.i32(5, c.E), c.i32(6, c.E + 1),
                   c.i32(7, c.A), c.i32(8, c.A), c.i32(9, c.S + 1), c.act(10, c.A * c.d), c.ws(11)};
  return c(g.symi_dispatch_capacity, v);
}
DEF(symi_dispatch_bwd) {
  Call c(a, n, 4);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.A * c.d), c.i32(2, c.A), c.act(3, c.T * c.d)};
  return c(g.symi_dispatch_bwd, v);
}
DEF(symi_expert_fwd) {
  Call c(a, n, 9);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.A * c.d), c.i32(2, c.S + 1), c.act(3, 2 * c.nw), c.act(4, c.nw), c.act(5, c.A * 2 * c.f),
                   c.act(6, c.A * c.f), c.act(7, c.A * c.d), c.ws(8)};
  return c(g.symi_expert_fwd, v);
}
template <class Fn>
PyObject* expert_bwd(Fn fn, PyObject* const* a, Py_ssize_t n, bool slots) {
  Call c(a, n, 13);
  if (!c.ok) Py_RETURN_NONE;
  const long long ng = slots ? c.nw : c.ne;
  const Val v[] = {c.act(1, c.A * c.d), c.act(2, c.A * c.d), c.act(3, c.A * 2 * c.f), c.act(4, c.A * c.f),
                   c.i32(5, c.S + 1), c.i32(6, c.E + 1), c.act(7, 2 * c.nw), c.act(8, c.nw), c.act(9, c.A * c.d),
                   c.f32(10, 2 * ng), c.f32(11, ng), c.ws(12)};
  return c(fn, v);
}
DEF(symi_expert_bwd) { return expert_bwd(g.symi_expert_bwd, a, n, false); }
DEF(symi_expert_bwd_active) { return expert_bwd(g.symi_expert_bwd_active, a, n, false); }
DEF(symi_expert_bwd_slots) { return expert_bwd(g.symi_expert_bwd_slots, a, n, true); }
DEF(symi_replica_allreduce) {
  Call c(a, n, 5);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.i32(1, c.E + 1), c.real(2), c.f32(3, 2 * c.nw), c.f32(4, c.nw)};
  return c(g.symi_replica_allreduce, v);
}
DEF(symi_router_fwd) {
  Call c(a, n, 5);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.T * c.d), c.act(2, c.E * c.d), c.f32_or_none(3, c.E), c.f32(4, c.T * c.E)};
  return c(g.symi_router_fwd, v);
}
DEF(symi_router_bwd) {
  Call c(a, n, 8);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.T * c.d), c.act(2, c.E * c.d), c.f32(3, c.T * c.E), c.f32(4, c.E * c.d),
                   c.f32_or_none(5, c.E), c.act(6, c.T * c.d), c.ws(7)};
  return c(g.symi_router_bwd, v);
}
DEF(symi_combine) {
  Call c(a, n, 5);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.A * c.d), c.i32(2, c.A), c.f32(3, c.A), c.act(4, c.T * c.d)};
  return c(g.symi_combine, v);
}
DEF(symi_combine_bwd) {
  Call c(a, n, 7);
  if (!c.ok) Py_RETURN_NONE;
  const Val v[] = {c.act(1, c.T * c.d), c.act(2, c.A * c.d), c.i32(3, c.A), c.f32(4, c.A), c.act(5, c.A * c.d),
                   c.f32(6, c.A)};
  return c(g.symi_combine_bwd, v);
}
// elements of one tensor of the optimizer's state: E shards of 3 d f / N
long long shard_state(const Call& c) { return c.E * (3 * c.d * c.f / c.c.N); }
DEF(symi_adam_to_replicas) {
  Call c(a, n, 10);
  if (!c.ok || c.c.N < 1) Py_RETURN_NONE;
  const long long per = shard_state(c);
  const Val v[] = {c.adam(1), c.f32(2, 2 * c.ne), c.f32(3, c.ne), c.f32(4, per), c.f32(5, per), c.f32(6, per),
                   c.i32(7, c.E + 1), c.act(8, 2 * c.nw), c.act(9, c.nw)};
  return c(g.symi_adam_to_replicas, v);
}
DEF(symi_adam_to_replicas_active) {
  Call c(a, n, 12);
  if (!c.ok || c.c.N < 1) Py_RETURN_NONE;
  const long long per = shard_state(c);
  const Val v[] = {c.adam(1), c.f32(2, 2 * c.ne), c.f32(3, c.ne), c.f32(4, per), c.f32(5, per), c.f32(6, per),
                   c.i32(7, c.S + 1), c.i32(8, c.E + 1), c.i32(9, c.E + 1), c.act(10, 2 * c.nw), c.act(11, c.nw)};
  return c(g.symi_adam_to_replicas_active, v);
}

// attach({name: address}, SymiCtx, SymiAdam)
PyObject* attach(PyObject*, PyObject* args) {
  PyObject *addresses, *ctx_type, *adam_type;
  if (!PyArg_ParseTuple(args, "O!O!O!", &PyDict_Type, &addresses, &PyType_Type, &ctx_type, &PyType_Type, &adam_type))
    return nullptr;
  Entries e;
#define X(name)                                                                       \
  {                                                                                   \
    PyObject* o = PyDict_GetItemString(addresses, #name);                             \
    void* p = o ? PyLong_AsVoidPtr(o) : nullptr;                                      \
    if (!p) {                                                                         \
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);                  \
      return nullptr;                                                                 \
    }                                                                                 \
    e.name = reinterpret_cast<decltype(&::name)>(p);                                  \
  }
  SYMI_CALLS(X)
#undef X
  Py_INCREF(ctx_type);
  Py_INCREF(adam_type);
  g_ctx_type = reinterpret_cast<PyTypeObject*>(ctx_type);
  g_adam_type = reinterpret_cast<PyTypeObject*>(adam_type);
  g = e;
  Py_RETURN_NONE;
}

#define M(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {
    M(symi_route) M(symi_route_bwd) M(symi_place) M(symi_dispatch) M(symi_dispatch_noalloc) M(symi_dispatch_capacity)
    M(symi_dispatch_bwd) M(symi_expert_fwd) M(symi_expert_bwd) M(symi_expert_bwd_slots) M(symi_expert_bwd_active)
    M(symi_replica_allreduce) M(symi_router_fwd) M(symi_router_bwd) M(symi_combine) M(symi_combine_bwd)
    M(symi_adam_to_replicas) M(symi_adam_to_replicas_active)
    {"attach", attach, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  g_ptr = PyUnicode_InternFromString("ptr");
  g_cfg = PyUnicode_InternFromString("cfg");
  if (!g_ptr || !g_cfg) return nullptr;
  return PyModule_Create(&module);
}
