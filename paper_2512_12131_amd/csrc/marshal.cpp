// Argument marshalling of the calls that small shapes make often, as a CPython module: output and workspace tensors, device
// pointers, sizes and the current stream, then the C ABI of lrboost.h.  No arithmetic and no state.
//
// Bound: host time.  A layer's forward and backward on a few hundred tokens are four launches of 3 us of host time each; the same
// marshalling through ctypes and torch's Python functions took another 18 us (1.7 us for each of seven tensors, 2-3 us for each
// call's twenty arguments), more than the GPU needs for the kernels.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include "lrboost.h"

namespace {

struct PyError {};   // a Python exception is set
PyObject* g_lr_error = nullptr;

[[noreturn]] void fail(PyObject* type, const char* what) {
  PyErr_SetString(type, what);
  throw PyError{};
}

// Positional arguments of a call.
struct Args {
  PyObject* const* v;
  Py_ssize_t n;
  Py_ssize_t at = 0;
  PyObject* next() {
    if (at >= n) fail(PyExc_TypeError, "too few arguments");
    return v[at++];
  }
  const at::Tensor& tensor() {
    PyObject* o = next();
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "tensor expected");
    return THPVariable_Unpack(o);
  }
  at::Tensor optional() { return at < n && v[at] == Py_None ? (at++, at::Tensor()) : tensor(); }
  int64_t integer() {
    PyObject* o = PyNumber_Index(next());
    if (!o) throw PyError{};
    const long long x = PyLong_AsLongLong(o);
    Py_DECREF(o);
    if (x == -1 && PyErr_Occurred()) throw PyError{};
    return x;
  }
  int enumerator() {
    const int64_t x = integer();
    if (x < INT_MIN || x > INT_MAX) fail(PyExc_OverflowError, "integer out of range");
    return (int)x;
  }
  float real() {
    const double x = PyFloat_AsDouble(next());
    if (x == -1.0 && PyErr_Occurred()) throw PyError{};
    return (float)x;
  }
};

int dt_of(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return LR_F32;
  if (t.scalar_type() == at::kBFloat16) return LR_BF16;
  fail(g_lr_error, "unsupported dtype");
}
at::ScalarType scalar(int dt) { return dt == LR_F32 ? at::kFloat : at::kBFloat16; }
int64_t rows_of(const at::Tensor& t, int dims = 2) {
  if (t.dim() != dims) fail(PyExc_ValueError, "unexpected number of dimensions");
  return t.size(0);
}
int64_t stride_of(const at::Tensor& t) {
  if (t.dim() != 2 || t.stride(1) != 1) fail(PyExc_AssertionError, "row-major 2-D tensor expected");
  return t.stride(0);
}
// The row stride of t, passed for the others too (of a single row any will do; beside a dense t, dense others of as many elements are the
// same rows in any shape).
int64_t stride_of_all(const at::Tensor& t, std::initializer_list<const at::Tensor*> others) {
  const int64_t ld = stride_of(t);
  for (const at::Tensor* o : others) {
    if ((ld == t.size(1) || t.size(0) <= 1) && o->is_contiguous() && o->numel() == t.numel()) continue;
    if (stride_of(*o) != ld && (t.size(0) > 1 || o->size(0) > 1)) fail(PyExc_AssertionError, "operands with the same row stride expected");
  }
  return ld;
}
int64_t size_of(const at::Tensor& t, int64_t i) {
  if (t.dim() <= i) fail(PyExc_IndexError, "tuple index out of range");
  return t.size(i);
}
void* ptr(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
// of an operand that no stride is passed for
void* dense(const at::Tensor& t) {
  if (t.defined() && !t.is_contiguous()) fail(PyExc_AssertionError, "contiguous tensor expected");
  return ptr(t);
}
at::Tensor fresh(at::IntArrayRef sizes, at::ScalarType dt, const at::Tensor& like) {
  return at::empty(sizes, at::TensorOptions().dtype(dt).device(like.device()));
}
// an output that is written with the row stride of t
at::Tensor rows_like(const at::Tensor& t) { return at::empty_strided(t.sizes(), t.strides(), t.options()); }
at::Tensor workspace(size_t bytes, const at::Tensor& like) {
  return fresh({(int64_t)(bytes < 256 ? 256 : bytes)}, at::kByte, like);
}
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// The call itself runs without the interpreter's lock.
template <class F>
void call(const char* what, F&& f) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = f();
  Py_END_ALLOW_THREADS
  if (status == LR_OK) return;
  PyErr_Format(g_lr_error, "%s failed: %s", what, lr_status_string(status));
  throw PyError{};
}

template <class... T>
PyObject* tuple(const T&... t) {
  PyObject* out = PyTuple_New(sizeof...(t));
  if (!out) throw PyError{};
  Py_ssize_t i = 0;
  for (const at::Tensor* x : {&t...}) {
    PyObject* o = THPVariable_Wrap(*x);
    if (!o) {
      Py_DECREF(out);
      throw PyError{};
    }
    PyTuple_SET_ITEM(out, i++, o);
  }
  return out;
}
PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }

// ---- one bottleneck layer ------------------------------------------------------------------
PyObject* linear_fwd(Args& a) {
  const at::Tensor &x = a.tensor(), &wd = a.tensor(), &wu = a.tensor();
  const int act = a.enumerator(), dt = dt_of(x);
  const int64_t T = rows_of(x), d = x.size(1), r = size_of(wd, 0), n = size_of(wu, 0);
  const at::Tensor z = fresh({T, r}, x.scalar_type(), x), y = fresh({T, n}, x.scalar_type(), x);
  const size_t nb = lr_linear_workspace_bytes(T, d, r, n, dt, 0);
  const at::Tensor ws = workspace(nb, x);
  const int64_t ldx = stride_of(x);
  void *px = ptr(x), *pd = dense(wd), *pu = dense(wu), *pz = ptr(z), *py = ptr(y), *pw = ptr(ws), *st = stream();
  call("lr_linear_fwd", [&] { return lr_linear_fwd(px, ldx, pd, pu, pz, py, n, T, d, r, n, act, dt, pw, nb, st); });
  return tuple(z, y);
}

PyObject* linear_fwd_static(Args& a) {
  const at::Tensor &x = a.tensor(), &wd = a.tensor(), &wu = a.tensor(), &z = a.tensor(), &y = a.tensor();
  const int act = a.enumerator();
  const int64_t T = rows_of(x), d = x.size(1), r = size_of(wd, 0), n = size_of(wu, 0);
  const int64_t zs[] = {T, r}, ys[] = {T, n};
  if (z.sizes() != at::IntArrayRef(zs) || y.sizes() != at::IntArrayRef(ys) || !z.is_contiguous() || !y.is_contiguous())
    fail(PyExc_AssertionError, "contiguous z [T, r] and y [T, d_out] expected");
  const int64_t ldx = stride_of(x);
  const int dt = dt_of(x);
  void *px = ptr(x), *pd = dense(wd), *pu = dense(wu), *pz = ptr(z), *py = ptr(y), *st = stream();
  call("lr_linear_fwd_static", [&] { return lr_linear_fwd_static(px, ldx, pd, pu, pz, py, n, T, d, r, n, act, dt, st); });
  return tuple(z, y);
}

PyObject* linear_bwd(Args& a) {
  const at::Tensor &x = a.tensor(), &wd = a.tensor(), &wu = a.tensor(), &z = a.tensor(), &dy = a.tensor();
  const int act = a.enumerator();
  const int acc = a.enumerator();
  at::Tensor dwd = a.optional(), dwu = a.optional();     // acc: added to
  const int gdt = a.enumerator(), dt = dt_of(x);
  const int64_t T = rows_of(x), d = x.size(1), r = size_of(wd, 0), n = size_of(wu, 0);
  const at::Tensor dx = fresh({T, d}, x.scalar_type(), x);
  if (!acc) {
    dwd = at::empty_like(wd, at::TensorOptions().dtype(scalar(gdt)));
    dwu = at::empty_like(wu, at::TensorOptions().dtype(scalar(gdt)));
  }
  const size_t nb = lr_linear_workspace_bytes(T, d, r, n, dt, 1);
  const at::Tensor ws = workspace(nb, x);
  const int64_t ldx = stride_of(x), lddy = stride_of(dy);
  void *px = ptr(x), *pd = dense(wd), *pu = dense(wu), *pz = dense(z), *py = ptr(dy), *pdx = ptr(dx), *gd = dense(dwd), *gu = dense(dwu),
       *pw = ptr(ws), *st = stream();
  call("lr_linear_bwd", [&] { return lr_linear_bwd(px, ldx, pd, pu, pz, py, lddy, pdx, d, gd, gu, T, d, r, n, act, dt, gdt, acc, pw, nb, st); });
  return tuple(dx, dwd, dwu);
}

// ---- G projections sharing one input ---------------------------------------------------------
PyObject* group_fwd(Args& a) {
  const at::Tensor& x = a.tensor();
  const at::Tensor gamma = a.optional();
  const float eps = a.real();
  const int norm = a.enumerator();
  const at::Tensor &wd = a.tensor(), &wu = a.tensor();
  const int act = a.enumerator(), dt = dt_of(x);
  const int64_t T = rows_of(x), d = x.size(1), G = rows_of(wu, 3), n = wu.size(1), r = wu.size(2);
  const at::Tensor z = fresh({T, G * r}, x.scalar_type(), x), stat = fresh({T}, at::kFloat, x), y = fresh({G, T, n}, x.scalar_type(), x);
  const size_t nb = lr_group_workspace_bytes((int)G, T, d, r, n, dt, 0);
  const at::Tensor ws = workspace(nb, x);
  const int64_t ldx = stride_of(x);
  void *px = ptr(x), *pg = dense(gamma), *pd = dense(wd), *pu = dense(wu), *pz = ptr(z), *ps = dense(stat), *py = ptr(y), *pw = ptr(ws), *st = stream();
  call("lr_group_fwd", [&] {
    return lr_group_fwd(px, ldx, pg, eps, norm, pd, pu, pz, (float*)ps, py, n, T * n, (int)G, T, d, r, n, act, dt, pw, nb, st);
  });
  return tuple(z, stat, y);
}

PyObject* group_bwd(Args& a) {
  const at::Tensor& x = a.tensor();
  const at::Tensor gamma = a.optional();
  const float eps = a.real();
  const int norm = a.enumerator();
  const at::Tensor &wd = a.tensor(), &wu = a.tensor(), &z = a.tensor();
  const at::Tensor stat = a.optional();
  const at::Tensor& dy = a.tensor();
  const int act = a.enumerator();
  const int acc = a.enumerator();
  at::Tensor dgamma = a.optional(), dwd = a.optional(), dwu = a.optional();   // acc: added to
  const int gdt = a.enumerator(), dt = dt_of(x);
  const int64_t T = rows_of(x), d = x.size(1), G = rows_of(wu, 3), n = wu.size(1), r = wu.size(2);
  const at::Tensor dx = fresh({T, d}, x.scalar_type(), x);
  if (!acc) {
    dgamma = fresh({d}, scalar(gdt), x);
    dwd = at::empty_like(wd, at::TensorOptions().dtype(scalar(gdt)));
    dwu = at::empty_like(wu, at::TensorOptions().dtype(scalar(gdt)));
  }
  const size_t nb = lr_group_workspace_bytes((int)G, T, d, r, n, dt, 1);
  const at::Tensor ws = workspace(nb, x);
  const int64_t ldx = stride_of(x);
  void *px = ptr(x), *pg = dense(gamma), *pd = dense(wd), *pu = dense(wu), *pz = dense(z), *ps = dense(stat), *py = dense(dy), *pdx = ptr(dx),
       *gg = dense(dgamma), *gd = dense(dwd), *gu = dense(dwu), *pw = ptr(ws), *st = stream();
  call("lr_group_bwd", [&] {
    return lr_group_bwd(px, ldx, pg, eps, norm, pd, pu, pz, (const float*)ps, py, n, T * n, pdx, d, gg, gd, gu, (int)G, T, d, r, n, act, dt, gdt,
                        acc, pw, nb, st);
  });
  return tuple(dx, dgamma, dwd, dwu);
}

// ---- attention -----------------------------------------------------------------------------
int64_t stride_of_kv(const at::Tensor& k, const at::Tensor& v) {
  const int64_t ldkv = stride_of(k);
  if (ldkv != stride_of(v)) fail(PyExc_AssertionError, "k and v with the same row stride expected");
  return ldkv;
}

PyObject* attention_fwd(Args& a) {
  const at::Tensor &q = a.tensor(), &k = a.tensor(), &v = a.tensor();
  const int64_t B = a.integer(), S = a.integer(), H = a.integer(), Hkv = a.integer(), hd = a.integer();
  const int causal = a.enumerator();
  const int64_t ld = stride_of(q), ldkv = stride_of_kv(k, v);
  const int dt = dt_of(q);
  const at::Tensor o = rows_like(q), lse = fresh({B, H, S}, at::kFloat, q);
  void *pq = ptr(q), *pk = ptr(k), *pv = ptr(v), *po = ptr(o), *pl = dense(lse), *st = stream();
  call("lr_attention_gqa_fwd", [&] { return lr_attention_gqa_fwd(pq, pk, pv, po, (float*)pl, ld, ldkv, B, S, H, Hkv, hd, causal, dt, st); });
  return tuple(o, lse);
}

PyObject* attention_bwd(Args& a) {
  const at::Tensor &q = a.tensor(), &k = a.tensor(), &v = a.tensor(), &o = a.tensor(), &dout = a.tensor(), &lse = a.tensor();
  const int64_t B = a.integer(), S = a.integer(), H = a.integer(), Hkv = a.integer(), hd = a.integer();
  const int causal = a.enumerator();
  const int64_t ld = stride_of_all(q, {&o, &dout}), ldkv = stride_of_kv(k, v);
  const at::Tensor dq = rows_like(q), dk = rows_like(k), dv = rows_like(k);
  const at::Tensor ws = workspace(lr_attention_gqa_bwd_workspace_bytes(B, S, H, Hkv, hd), q);
  const size_t nb = (size_t)ws.numel();
  const int dt = dt_of(q);
  void *pq = ptr(q), *pk = ptr(k), *pv = ptr(v), *po = ptr(o), *pdo = ptr(dout), *pl = dense(lse), *gq = ptr(dq), *gk = ptr(dk), *gv = ptr(dv),
       *pw = ptr(ws), *st = stream();
  call("lr_attention_gqa_bwd", [&] {
    return lr_attention_gqa_bwd(pq, pk, pv, po, pdo, (const float*)pl, gq, gk, gv, ld, ldkv, B, S, H, Hkv, hd, causal, dt, pw, nb, st);
  });
  return tuple(dq, dk, dv);
}

// ---- standalone memory-bound kernels ---------------------------------------------------------
PyObject* rms_stat(Args& a) {
  const at::Tensor& x = a.tensor();
  const int64_t T = rows_of(x), d = x.size(1);
  const at::Tensor stat = fresh({T}, at::kFloat, x);
  const int64_t ldx = stride_of(x);
  const int dt = dt_of(x);
  void *px = ptr(x), *ps = dense(stat), *st = stream();
  call("lr_rms_stat", [&] { return lr_rms_stat(px, ldx, (float*)ps, T, d, dt, st); });
  return wrap(stat);
}

PyObject* rmsnorm_apply(Args& a) {
  const at::Tensor &x = a.tensor(), &gamma = a.tensor(), &stat = a.tensor();
  const float eps = a.real();
  const int64_t T = rows_of(x), d = x.size(1);
  const at::Tensor out = at::empty_like(x);
  const int64_t ldx = stride_of(x);
  const int dt = dt_of(x);
  void *px = ptr(x), *pg = dense(gamma), *ps = dense(stat), *po = ptr(out), *st = stream();
  call("lr_rmsnorm_apply", [&] { return lr_rmsnorm_apply(px, ldx, pg, (const float*)ps, eps, po, d, T, d, dt, st); });
  return wrap(out);
}

PyObject* rmsnorm_bwd(Args& a) {
  const at::Tensor &x = a.tensor(), &gamma = a.tensor(), &stat = a.tensor();
  const float eps = a.real();
  const at::Tensor& dxhat = a.tensor();
  const at::Tensor dres = a.optional();
  const int64_t T = rows_of(x), d = x.size(1);
  const at::Tensor dx = at::empty_like(x);
  const int64_t parts = lr_rmsnorm_bwd_parts(T);
  const at::Tensor part = fresh({parts < 1 ? 1 : parts, d}, at::kFloat, x);
  const int64_t ldx = stride_of(x), lddxh = stride_of(dxhat), lddres = dres.defined() ? stride_of(dres) : 0;
  const int dt = dt_of(x);
  void *px = ptr(x), *pg = dense(gamma), *ps = dense(stat), *ph = ptr(dxhat), *pr = ptr(dres), *pdx = ptr(dx), *pp = ptr(part), *st = stream();
  call("lr_rmsnorm_bwd", [&] { return lr_rmsnorm_bwd(px, ldx, pg, (const float*)ps, eps, ph, lddxh, pr, lddres, pdx, d, (float*)pp, T, d, dt, st); });
  return tuple(dx, part);
}

PyObject* swiglu_fwd(Args& a) {
  const at::Tensor &g = a.tensor(), &u = a.tensor();
  const int64_t T = rows_of(g), f = g.size(1);
  const int64_t ld = stride_of_all(g, {&u});
  const at::Tensor m = rows_like(g);
  const int dt = dt_of(g);
  void *pg = ptr(g), *pu = ptr(u), *pm = ptr(m), *st = stream();
  call("lr_swiglu_fwd", [&] { return lr_swiglu_fwd(pg, pu, pm, ld, T, f, dt, st); });
  return wrap(m);
}

PyObject* swiglu_bwd(Args& a) {
  const at::Tensor &g = a.tensor(), &u = a.tensor(), &dm = a.tensor();
  const int64_t T = rows_of(g), f = g.size(1);
  const int64_t ld = stride_of_all(g, {&u, &dm});
  const at::Tensor dg = rows_like(g), du = rows_like(u);
  const int dt = dt_of(g);
  void *pg = ptr(g), *pu = ptr(u), *pm = ptr(dm), *gg = ptr(dg), *gu = ptr(du), *st = stream();
  call("lr_swiglu_bwd", [&] { return lr_swiglu_bwd(pg, pu, pm, gg, gu, ld, T, f, dt, st); });
  return tuple(dg, du);
}

// No C++ exception leaves an entry; torch's own become the Python exceptions that they are elsewhere (out of memory, a device's error,
// an interpreter's exception that crossed torch).
template <PyObject* (*F)(Args&)>
PyObject* entry(PyObject*, PyObject* const* v, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  try {
    Args a{v, n};
    return F(a);
  } catch (const PyError&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

PyObject* set_error(PyObject*, PyObject* type) {
  Py_INCREF(type);
  Py_XSETREF(g_lr_error, type);
  Py_RETURN_NONE;
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))(&entry<f>), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    ENTRY(linear_fwd), ENTRY(linear_fwd_static), ENTRY(linear_bwd), ENTRY(group_fwd), ENTRY(group_bwd), ENTRY(attention_fwd), ENTRY(attention_bwd),
    ENTRY(rms_stat), ENTRY(rmsnorm_apply), ENTRY(rmsnorm_bwd), ENTRY(swiglu_fwd), ENTRY(swiglu_bwd),
    {"set_error", set_error, METH_O, "the exception type of failed calls"}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  PyObject* m = PyModule_Create(&g_module);
  if (m) {
    Py_INCREF(PyExc_RuntimeError);
    g_lr_error = PyExc_RuntimeError;
  }
  return m;
}
