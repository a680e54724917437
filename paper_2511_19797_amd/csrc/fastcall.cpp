// The binding's ordinary calls in native code: argument checks, outputs and workspace, descriptor, the library's entry point.
//
// Small calls are bound by the host: two attention calls of three kernels (20 us on the GPU) took 47 us, the eleven calls of a
// block's forward on one image (100 us of kernels) 161 us, most of it ctypes, torch's Python layer and tuples of shapes.
// Every function here takes the arguments of the binding's function of the same name (binding.py), does exactly what that does
// for plain tensors that pass its checks, and returns None, before anything has happened, for whatever else: binding.py then
// goes its own way, which raises where it always did.  A failing entry point returns its status (an int).
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <limits>

#include "../../include/tvmattn.h"

namespace {

using at::Tensor;

// An argument as a plain strided tensor on the GPU, or nothing.  (Transforms, subclasses, lazily conjugated or negated views:
// binding.py's way.)
const Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
  const auto ks = t.key_set();
  using K = c10::DispatchKey;
  if (ks.has(K::Python) || ks.has(K::FuncTorchBatched) || ks.has(K::FuncTorchGradWrapper) || ks.has(K::Functionalize) ||
      ks.has(K::Conjugate) || ks.has(K::Negative) || ks.has(K::ZeroTensor))
    return nullptr;
  return &t;
}

// No mode or transform is active that would see, or replace, the tensors made here.
bool ordinary() {
  return !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled() &&
         !c10::impl::tls_local_dispatch_key_set().included_.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

// Positional arguments: required tensors, optional ones (None), numbers.
struct Args {
  PyObject* const* a;
  Py_ssize_t n;
  bool ok = ordinary();
  const Tensor* t(Py_ssize_t i) {
    const Tensor* p = i < n ? plain(a[i]) : nullptr;
    if (p == nullptr) ok = false;
    return p;
  }
  const Tensor* opt(Py_ssize_t i) { return i < n && a[i] == Py_None ? nullptr : t(i); }
  double f(Py_ssize_t i) {
    if (i >= n || !(PyFloat_Check(a[i]) || PyLong_Check(a[i]))) return ok = false, 0.0;
    const double v = PyFloat_AsDouble(a[i]);
    if (v == -1.0 && PyErr_Occurred()) return PyErr_Clear(), ok = false, 0.0;
    return v;
  }
  bool flag(Py_ssize_t i) {
    if (i >= n || !PyBool_Check(a[i])) return ok = false, false;
    return a[i] == Py_True;
  }
  int32_t whole(Py_ssize_t i) {
    if (i >= n || !PyLong_Check(a[i])) return ok = false, 0;
    const long v = PyLong_AsLong(a[i]);
    if ((v == -1 && PyErr_Occurred()) || v < INT32_MIN || v > INT32_MAX) return PyErr_Clear(), ok = false, 0;
    return (int32_t)v;
  }
};

bool same_layout(const Tensor& r, const Tensor* t) {
  return t == nullptr || (t->scalar_type() == r.scalar_type() && t->device() == r.device() && t->sizes() == r.sizes() &&
                          t->strides() == r.strides());
}
template <class... Ts>
bool same_layouts(const Tensor& r, Ts... ts) {
  return (same_layout(r, ts) && ...);
}
bool small(int64_t v) { return v <= std::numeric_limits<int32_t>::max(); }

bool type_of(const Tensor& t, int32_t& dt) {
  if (t.scalar_type() == at::kFloat) dt = TVMATTN_F32;
  else if (t.scalar_type() == at::kBFloat16) dt = TVMATTN_BF16;
  else return false;
  return true;
}
bool make_desc(tvmattn_desc& d, const Tensor& k, const Tensor& q, double scale, int32_t flags) {
  if (k.dim() != 4 || q.dim() != 4 || k.stride(3) != 1 || q.stride(3) != 1) return false;
  if (q.scalar_type() != k.scalar_type() || q.size(0) != k.size(0) || q.size(1) != k.size(1) || q.size(3) != k.size(3)) return false;
  for (int i = 0; i < 4; ++i)
    if (!small(k.size(i)) || !small(q.size(i))) return false;
  d = tvmattn_desc{};
  if (!type_of(k, d.dtype)) return false;
  d.B = (int32_t)k.size(0);
  d.H = (int32_t)k.size(1);
  d.N = (int32_t)k.size(2);
  d.D = (int32_t)k.size(3);
  d.scale = (float)scale;
  d.stride_b = k.stride(0);
  d.stride_h = k.stride(1);
  d.stride_n = k.stride(2);
  d.M = (int32_t)q.size(2);
  d.flags = flags;
  d.qstride_b = q.stride(0);
  d.qstride_h = q.stride(1);
  d.qstride_n = q.stride(2);
  return true;
}

Tensor like(const Tensor& r) { return at::empty_strided(r.sizes(), r.strides(), r.options()); }
Tensor row_vector(const Tensor& q) { return at::empty({q.size(0), q.size(1), q.size(2)}, q.options().dtype(at::kFloat)); }
Tensor bytes(const Tensor& r, size_t n) { return at::empty({(int64_t)n}, r.options().dtype(at::kByte)); }
void* ptr(const Tensor* t) { return t == nullptr ? nullptr : t->data_ptr(); }
void* ptr(const Tensor& t) { return t.data_ptr(); }
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// An entry point with the interpreter released: it never touches Python objects.  Its arguments are raw pointers and numbers,
// worked out before: a data pointer may throw (storages that refuse access) or copy a storage (copy-on-write), and that has to
// happen while the interpreter is held.
template <class... P, class... A>
int released(int (*entry)(P...), A... a) {
  int rc;
  Py_BEGIN_ALLOW_THREADS rc = entry(a...);
  Py_END_ALLOW_THREADS
  return rc;
}
// The outputs as a tuple (an undefined tensor is None), or the status.
template <size_t N>
PyObject* result(int rc, const Tensor (&t)[N]) {
  if (rc != 0) return PyLong_FromLong(rc);
  PyObject* r = PyTuple_New(N);
  if (r == nullptr) return nullptr;
  for (size_t i = 0; i < N; ++i) {
    PyObject* o = t[i].defined() ? THPVariable_Wrap(t[i]) : Py_NewRef(Py_None);
    if (o == nullptr) {
      Py_DECREF(r);
      return nullptr;
    }
    PyTuple_SET_ITEM(r, i, o);
  }
  return r;
}
// No C++ exception leaves a function: torch's become Python's, as in torch's own functions (out of memory above all).
template <class F>
PyObject* guarded(F&& f) {
  HANDLE_TH_ERRORS
  return f();
  END_HANDLE_TH_ERRORS
}
#define NOT_MINE Py_RETURN_NONE

// q k v tq tk tv scale save flags
PyObject* jvp_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *q = g.t(0), *k = g.t(1), *v = g.t(2), *tq = g.t(3), *tk = g.t(4), *tv = g.t(5);
    const double scale = g.f(6);
    const bool save = g.flag(7);
    const int32_t flags = g.whole(8);
    tvmattn_desc d;
    if (!g.ok || !same_layout(*q, tq) || !same_layouts(*k, v, tk, tv) || q->device() != k->device() || !make_desc(d, *k, *q, scale, flags))
      NOT_MINE;
    Tensor o[4] = {like(*q), like(*q)};
    if (save) o[2] = row_vector(*q), o[3] = row_vector(*q);
    void* const st = stream();
    const int rc = released(tvmattn_jvp_fwd, &d, ptr(q), ptr(k), ptr(v), ptr(tq), ptr(tk), ptr(tv), ptr(o[0]), ptr(o[1]),
                            save ? (float*)ptr(o[2]) : nullptr, save ? (float*)ptr(o[3]) : nullptr, st);
    return result(rc, o);
  });
}

// q k v tq tk tv o to lse stats gO gTO scale flags
PyObject* jvp_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *q = g.t(0), *k = g.t(1), *v = g.t(2), *tq = g.opt(3), *tk = g.opt(4), *tv = g.opt(5), *o = g.t(6), *to = g.opt(7),
                 *lse = g.t(8), *stats = g.opt(9), *gO = g.opt(10), *gTO = g.opt(11);
    const double scale = g.f(12);
    const int32_t flags = g.whole(13);
    tvmattn_desc d;
    if (!g.ok || !same_layouts(*q, tq, o, to, gO, gTO) || !same_layouts(*k, v, tk, tv) || q->device() != k->device() ||
        !make_desc(d, *k, *q, scale, flags))
      NOT_MINE;
    Tensor r[6] = {like(*q), like(*k), like(*k)};  // dq, dk, dv, dtq, dtk, dtv
    if (gTO != nullptr) r[3] = like(*q), r[4] = like(*k), r[5] = like(*k);
    const size_t need = tvmattn_jvp_bwd_workspace_bytes(&d);
    const Tensor ws = bytes(*q, need);
    auto out = [&](int i) { return r[i].defined() ? ptr(r[i]) : nullptr; };
    void* const st = stream();
    const int rc = released(tvmattn_jvp_bwd, &d, ptr(q), ptr(k), ptr(v), ptr(tq), ptr(tk), ptr(tv), ptr(o), ptr(to),
                            (const float*)ptr(lse), (const float*)ptr(stats), ptr(gO), ptr(gTO), out(0), out(1), out(2), out(3),
                            out(4), out(5), ptr(ws), need, st);
    return result(rc, r);
  });
}

bool gain_ok(const Tensor& g, const Tensor& ref) {
  return g.scalar_type() == at::kFloat && g.dim() == 1 && g.size(0) == ref.size(3) && g.is_contiguous() && g.device() == ref.device();
}

// q tq k tk gain_q gain_k eps
PyObject* qknorm_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *q = g.t(0), *tq = g.t(1), *k = g.t(2), *tk = g.t(3), *gq = g.t(4), *gk = g.t(5);
    const double eps = g.f(6);
    tvmattn_desc d;
    if (!g.ok || !same_layout(*q, tq) || !same_layout(*k, tk) || q->device() != k->device() || !make_desc(d, *k, *q, 0.0, 0) ||
        !gain_ok(*gq, *q) || !gain_ok(*gk, *k))
      NOT_MINE;
    Tensor o[4] = {like(*q), like(*q), like(*k), like(*k)};
    void* const st = stream();
    const int rc = released(tvmattn_qknorm_jvp_fwd, &d, ptr(q), ptr(tq), ptr(k), ptr(tk), (const float*)ptr(gq),
                            (const float*)ptr(gk), (float)eps, ptr(o[0]), ptr(o[1]), ptr(o[2]), ptr(o[3]), st);
    return result(rc, o);
  });
}

// q tq k tk gain_q gain_k eps qn tqn kn tkn v tv o to lse stats gO gTO scale, then the six gradients and two gain gradients
PyObject* bwd_qknorm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *q = g.t(0), *tq = g.t(1), *k = g.t(2), *tk = g.t(3), *gq = g.t(4), *gk = g.t(5), *qn = g.t(7), *tqn = g.t(8),
                 *kn = g.t(9), *tkn = g.t(10), *v = g.t(11), *tv = g.t(12), *o = g.t(13), *to = g.t(14), *lse = g.t(15),
                 *stats = g.t(16), *gO = g.t(17), *gTO = g.t(18);
    const double eps = g.f(6), scale = g.f(19);
    const Tensor* r[8];
    for (int i = 0; i < 8; ++i) r[i] = g.t(20 + i);
    tvmattn_desc d;
    if (!g.ok || !same_layouts(*q, tq, qn, tqn, o, to, gO, gTO, r[0], r[3]) ||
        !same_layouts(*k, tk, kn, tkn, v, tv, r[1], r[2], r[4], r[5]) || q->device() != k->device() ||
        !make_desc(d, *k, *q, scale, 0) || !gain_ok(*gq, *q) || !gain_ok(*gk, *k) || !gain_ok(*r[6], *q) || !gain_ok(*r[7], *k))
      NOT_MINE;
    const size_t need = tvmattn_jvp_bwd_qknorm_workspace_bytes(&d), size = need > 16 ? need : 16;
    const Tensor ws = bytes(*q, size);
    void* const st = stream();
    const int rc = released(tvmattn_jvp_bwd_qknorm, &d, ptr(q), ptr(tq), ptr(k), ptr(tk), (const float*)ptr(gq),
                            (const float*)ptr(gk), (float)eps, ptr(qn), ptr(tqn), ptr(kn), ptr(tkn), ptr(v), ptr(tv), ptr(o),
                            ptr(to), (const float*)ptr(lse), (const float*)ptr(stats), ptr(gO), ptr(gTO), ptr(r[0]), ptr(r[1]),
                            ptr(r[2]), ptr(r[3]), ptr(r[4]), ptr(r[5]), (float*)ptr(r[6]), (float*)ptr(r[7]), ptr(ws), size, st);
    return PyLong_FromLong(rc);
  });
}

// x and its tangent: contiguous [B,T,C] of one type; the modulation vectors: contiguous float32 [B,C]
bool token_args(const Tensor& x, const Tensor& tx, std::initializer_list<const Tensor*> mods, int32_t& dt) {
  if (x.dim() != 3 || !x.is_contiguous() || tx.sizes() != x.sizes() || tx.scalar_type() != x.scalar_type() || !tx.is_contiguous()) return false;
  if (!small(x.size(0)) || !small(x.size(1)) || !small(x.size(2)) || !type_of(x, dt)) return false;
  for (const Tensor* m : mods)
    if (m->dim() != 2 || m->size(0) != x.size(0) || m->size(1) != x.size(2) || m->scalar_type() != at::kFloat || !m->is_contiguous() ||
        m->device() != x.device())
      return false;
  return true;
}
bool looks_like(const Tensor& x, const Tensor& u, const Tensor& tu) {
  return u.is_contiguous() && tu.is_contiguous() && u.sizes() == x.sizes() && tu.sizes() == x.sizes() && u.scalar_type() == x.scalar_type() &&
         tu.scalar_type() == x.scalar_type();
}
#define DIMS(x) (int)x->size(0), (int)x->size(1), (int)x->size(2)

// x tx a ta b tb eps
PyObject* adaln_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *x = g.t(0), *tx = g.t(1), *s = g.t(2), *ts = g.t(3), *b = g.t(4), *tb = g.t(5);
    const double eps = g.f(6);
    int32_t dt;
    if (!g.ok || !token_args(*x, *tx, {s, ts, b, tb}, dt)) NOT_MINE;
    Tensor o[2] = {like(*x), like(*x)};
    void* const st = stream();
    const int rc = released(tvmattn_adaln_jvp_fwd, DIMS(x), dt, ptr(x), ptr(tx), (const float*)ptr(s), (const float*)ptr(ts),
                            (const float*)ptr(b), (const float*)ptr(tb), (float)eps, ptr(o[0]), ptr(o[1]), st);
    return result(rc, o);
  });
}

// x tx a ta b tb eps gy gty gres gtres
PyObject* adaln_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *x = g.t(0), *tx = g.t(1), *s = g.t(2), *ts = g.t(3), *b = g.t(4), *tb = g.t(5), *gy = g.t(7), *gty = g.t(8),
                 *gres = g.opt(9), *gtres = g.opt(10);
    const double eps = g.f(6);
    int32_t dt;
    if (!g.ok || !token_args(*x, *tx, {s, ts, b, tb}, dt) || !looks_like(*x, *gy, *gty) || (gres == nullptr) != (gtres == nullptr) ||
        (gres != nullptr && !looks_like(*x, *gres, *gtres)))
      NOT_MINE;
    Tensor o[6] = {like(*x), like(*x), like(*s), like(*s), like(*s), like(*s)};
    const size_t need = tvmattn_adaln_jvp_bwd_workspace_bytes(DIMS(x), dt), size = need > 16 ? need : 16;
    const Tensor ws = bytes(*x, size);
    void* const st = stream();
    const int rc = released(tvmattn_adaln_jvp_bwd_residual, DIMS(x), dt, ptr(x), ptr(tx), (const float*)ptr(s),
                            (const float*)ptr(ts), (const float*)ptr(b), (const float*)ptr(tb), (float)eps, ptr(gy), ptr(gty),
                            ptr(gres), ptr(gtres), ptr(o[0]), ptr(o[1]), (float*)ptr(o[2]), (float*)ptr(o[3]), (float*)ptr(o[4]),
                            (float*)ptr(o[5]), ptr(ws), size, st);
    return result(rc, o);
  });
}

// x tx h th c tc eps
PyObject* gate_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *x = g.t(0), *tx = g.t(1), *h = g.t(2), *th = g.t(3), *c = g.t(4), *tc = g.t(5);
    const double eps = g.f(6);
    int32_t dt;
    if (!g.ok || !token_args(*x, *tx, {c, tc}, dt) || !looks_like(*x, *h, *th)) NOT_MINE;
    Tensor o[2] = {like(*x), like(*x)};
    void* const st = stream();
    const int rc = released(tvmattn_gate_jvp_fwd, DIMS(x), dt, ptr(x), ptr(tx), ptr(h), ptr(th), (const float*)ptr(c),
                            (const float*)ptr(tc), (float)eps, ptr(o[0]), ptr(o[1]), st);
    return result(rc, o);
  });
}

// h th c tc eps gz gtz
PyObject* gate_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *h = g.t(0), *th = g.t(1), *c = g.t(2), *tc = g.t(3), *gz = g.t(5), *gtz = g.t(6);
    const double eps = g.f(4);
    int32_t dt;
    if (!g.ok || !token_args(*h, *th, {c, tc}, dt) || !looks_like(*h, *gz, *gtz)) NOT_MINE;
    Tensor o[4] = {like(*h), like(*h), like(*c), like(*c)};
    const size_t need = tvmattn_gate_jvp_bwd_workspace_bytes(DIMS(h), dt), size = need > 16 ? need : 16;
    const Tensor ws = bytes(*h, size);
    void* const st = stream();
    const int rc = released(tvmattn_gate_jvp_bwd, DIMS(h), dt, ptr(h), ptr(th), (const float*)ptr(c), (const float*)ptr(tc),
                            (float)eps, ptr(gz), ptr(gtz), ptr(o[0]), ptr(o[1]), (float*)ptr(o[2]), (float*)ptr(o[3]), ptr(ws),
                            size, st);
    return result(rc, o);
  });
}

bool pointwise(const Tensor& f, std::initializer_list<const Tensor*> rest, int32_t& dt) {
  if (!f.is_contiguous() || !type_of(f, dt)) return false;
  for (const Tensor* t : rest)
    if (t->sizes() != f.sizes() || t->scalar_type() != f.scalar_type() || t->device() != f.device() || !t->is_contiguous()) return false;
  return true;
}
// u tu
PyObject* gelu_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *u = g.t(0), *tu = g.t(1);
    int32_t dt;
    if (!g.ok || !pointwise(*u, {tu}, dt)) NOT_MINE;
    Tensor o[2] = {like(*u), like(*u)};
    void* const st = stream();
    const int rc = released(tvmattn_gelu_jvp_fwd, u->numel(), dt, ptr(u), ptr(tu), ptr(o[0]), ptr(o[1]), st);
    return result(rc, o);
  });
}
// u tu ga gta
PyObject* gelu_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *u = g.t(0), *tu = g.t(1), *ga = g.t(2), *gta = g.t(3);
    int32_t dt;
    if (!g.ok || !pointwise(*u, {tu, ga, gta}, dt)) NOT_MINE;
    Tensor o[2] = {like(*u), like(*u)};
    void* const st = stream();
    const int rc = released(tvmattn_gelu_jvp_bwd, u->numel(), dt, ptr(u), ptr(tu), ptr(ga), ptr(gta), ptr(o[0]), ptr(o[1]), st);
    return result(rc, o);
  });
}

// A tensor as rows of `cols` elements: contiguous [..., cols], or a 2-D view with any row pitch.
bool rows(const Tensor& t, int64_t cols, int64_t& R, int64_t& ld) {
  if (t.dim() < 1 || t.size(-1) != cols || t.stride(-1) != 1) return false;
  if (t.is_contiguous()) {
    if (cols == 0) return false;
    R = t.numel() / cols, ld = cols;
  } else if (t.dim() == 2) {
    R = t.size(0), ld = t.stride(0);
  } else {
    return false;
  }
  return small(R);
}
bool linear_args(const Tensor& x, const Tensor& tx, const Tensor& w, const Tensor* bias, int64_t& R, int64_t& ldx, int32_t& dt) {
  if (w.dim() != 2 || w.scalar_type() != x.scalar_type() || !w.is_contiguous() || w.device() != x.device()) return false;
  if (!small(w.size(0)) || !small(w.size(1)) || !rows(x, w.size(1), R, ldx) || !same_layout(x, &tx) || !type_of(x, dt)) return false;
  return bias == nullptr || (bias->dim() == 1 && bias->size(0) == w.size(0) && bias->scalar_type() == x.scalar_type() &&
                             bias->is_contiguous() && bias->device() == x.device());
}
// x tx w bias
PyObject* linear_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *x = g.t(0), *tx = g.t(1), *w = g.t(2), *bias = g.opt(3);
    int64_t R, ldx;
    int32_t dt;
    if (!g.ok || !linear_args(*x, *tx, *w, bias, R, ldx, dt) || w->size(0) == 0) NOT_MINE;
    const int64_t F = w->size(0);
    auto shape = x->sizes().vec();
    shape.back() = F;
    Tensor o[2] = {at::empty(shape, x->options()), at::empty(shape, x->options())};
    void* const st = stream();
    const int rc = released(tvmattn_linear_jvp_fwd, (int)R, (int)w->size(1), (int)F, dt, ptr(x), ptr(tx), ldx, ptr(w), ptr(bias),
                            ptr(o[0]), ptr(o[1]), F, st);
    return result(rc, o);
  });
}
// x tx w gy gty bias_grad
PyObject* linear_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    Args g{a, n};
    const Tensor *x = g.t(0), *tx = g.t(1), *w = g.t(2), *gy = g.t(3), *gty = g.t(4);
    const bool bias_grad = g.flag(5);
    int64_t R, ldx, Ry, ldy;
    int32_t dt;
    if (!g.ok || !linear_args(*x, *tx, *w, nullptr, R, ldx, dt) || !rows(*gy, w->size(0), Ry, ldy) || Ry != R ||
        gty->sizes() != gy->sizes() || gty->strides() != gy->strides() || gy->scalar_type() != x->scalar_type() ||
        gty->scalar_type() != x->scalar_type())
      NOT_MINE;
    const int K = (int)w->size(1), F = (int)w->size(0);
    Tensor o[4] = {like(*x), like(*x), like(*w)};
    if (bias_grad) o[3] = at::empty({F}, x->options());
    const size_t need = tvmattn_linear_jvp_bwd_workspace_bytes((int)R, K, F, dt), size = need > 16 ? need : 16;
    const Tensor ws = bytes(*x, size);
    void* const st = stream();
    const int rc = released(tvmattn_linear_jvp_bwd, (int)R, K, F, dt, ptr(x), ptr(tx), ldx, ptr(w), ptr(gy), ptr(gty), ldy,
                            ptr(o[0]), ptr(o[1]), ptr(o[2]), bias_grad ? ptr(o[3]) : nullptr, ptr(ws), size, st);
    return result(rc, o);
  });
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(jvp_fwd),  METHOD(jvp_bwd),  METHOD(qknorm_fwd), METHOD(bwd_qknorm), METHOD(adaln_fwd), METHOD(adaln_bwd),
                         METHOD(gate_fwd), METHOD(gate_bwd), METHOD(gelu_fwd),   METHOD(gelu_bwd),   METHOD(linear_fwd), METHOD(linear_bwd),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and the Python that this was compiled against; binding.py uses the module with no other.
PyMODINIT_FUNC PyInit__fastcall() {
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", TVM_BUILT_FOR) != 0) Py_CLEAR(m);
  return m;
}
