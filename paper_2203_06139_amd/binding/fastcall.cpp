// fastcall.cpp -- native argument marshalling of the binding's per-call entry
// points (CPython extension module _fastcall).
//
// A call of the objective is one or two kernels of a few microseconds; taking
// its arguments apart in Python and through ctypes took 16 us, here it takes
// under 5.  Calls in a row, in us each, Python against this: gradient of 1000
// bins 15.6 against 5.7, of 1e5 bins in FP32 per bin 19.3 against 9.3,
// expected Hessian and covariance of 1e6 bins 29.7 against 16.2 (the kernels'
// own time in all three).
//
// Each function here takes the Python function's arguments, and where every
// tensor already is what the kernels need (plain tensors on one GPU, dtypes,
// contiguity, sizes) and the stream's context is known, it allocates the
// outputs, makes the C call and returns the Python function's result, or
// raises HistfitError with the library's message where the call fails.  In
// every other case (conversions, a first call on a stream, wrong arguments,
// active dispatch modes) it returns None and does nothing, and the Python code
// after it converts or raises.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <optional>

#include "../../include/histfit.h"

namespace {

struct Api {
  decltype(&::hf_model_nparams) nparams = nullptr;
  decltype(&::nll_eval) eval = nullptr;
  decltype(&::nll_grad) grad = nullptr;
  decltype(&::nll_unbinned) unbinned = nullptr;
  decltype(&::hf_nll_fisher) fisher = nullptr;
  decltype(&::hf_fisher_covariance) covariance = nullptr;
  decltype(&::fit_batch) fit = nullptr;
  decltype(&::hf_last_error) last_error = nullptr;
} api;
PyObject* error_type = nullptr;  // HistfitError

// The Python side's dictionaries: (device, stream) -> context, device -> list of
// spare contexts, of which a call outside capture keeps `spares`.  They are
// looked up on every call, so that there is one record of the contexts.
PyObject* contexts = nullptr;
PyObject* pools = nullptr;
Py_ssize_t spares = 0;

PyObject *s_counts, *s_weights, *s_edges, *s_xrange, *s_yrange, *s_kind, *s_n_gauss, *s_poly_degree,
    *s_t_shift, *s_t_scale, *s_bin_average, *s_value;

struct Owned {  // a new reference
  PyObject* o;
  explicit Owned(PyObject* p) : o(p) {}
  ~Owned() { Py_XDECREF(o); }
  Owned(const Owned&) = delete;
  Owned& operator=(const Owned&) = delete;
};

bool modes_active() {
  return c10::impl::TorchDispatchModeTLS::any_modes_set() ||
         at::impl::PythonTorchFunctionTLS::stack_len() > 0;
}

// o as a plain contiguous tensor of `type` on GPU `dev` (any GPU if dev < 0)
// with at least n values; null otherwise.
const at::Tensor* plain(PyObject* o, int dev, c10::ScalarType type, int64_t n) {
  if (!o || !THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  constexpr c10::DispatchKeySet wrapped =
      c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                           c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                           c10::DispatchKey::Negative, c10::DispatchKey::Conjugate,
                           c10::DispatchKey::ZeroTensor});
  if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || t.key_set().has_any(wrapped))
    return nullptr;
  if (dev >= 0 && t.get_device() != dev) return nullptr;
  if (t.scalar_type() != type || !t.is_contiguous() || t.numel() < n || !t.has_storage()) return nullptr;
  return &t;
}

bool is_none(PyObject* o) { return o == Py_None; }

// An optional output: the given tensor, or a new one shaped `sizes`.
struct Out {
  at::Tensor made;
  PyObject* given = nullptr;
  void* ptr = nullptr;
  bool take(PyObject* o, const at::Tensor& like, c10::ScalarType type, at::IntArrayRef sizes) {
    if (!is_none(o)) {
      const at::Tensor* t = plain(o, like.get_device(), type, c10::multiply_integers(sizes));
      if (!t) return false;
      given = o;
      ptr = t->data_ptr();
      return true;
    }
    made = at::empty(sizes, like.options().dtype(type).requires_grad(false));
    ptr = made.data_ptr();
    return true;
  }
  PyObject* wrap() {
    if (given) {
      Py_INCREF(given);
      return given;
    }
    return THPVariable_Wrap(std::move(made));
  }
};

bool to_int(PyObject* o, long* v) {
  if (!PyLong_Check(o)) return false;
  *v = PyLong_AsLong(o);
  return !(*v == -1 && PyErr_Occurred());
}
bool to_double(PyObject* o, double* v) {
  if (!PyFloat_Check(o) && !PyLong_Check(o)) return false;
  *v = PyFloat_AsDouble(o);
  return !(*v == -1.0 && PyErr_Occurred());
}
bool attr_int(PyObject* o, PyObject* name, int32_t* v) {
  Owned a(PyObject_GetAttr(o, name));
  long x;
  if (!a.o || !to_int(a.o, &x)) return false;
  *v = static_cast<int32_t>(x);
  return *v == x;
}
bool attr_double(PyObject* o, PyObject* name, double* v) {
  Owned a(PyObject_GetAttr(o, name));
  return a.o && to_double(a.o, v);
}
bool attr_range(PyObject* o, PyObject* name, double* lo, double* hi) {
  Owned a(PyObject_GetAttr(o, name));
  return a.o && PyTuple_Check(a.o) && PyTuple_GET_SIZE(a.o) >= 2 &&
         to_double(PyTuple_GET_ITEM(a.o, 0), lo) && to_double(PyTuple_GET_ITEM(a.o, 1), hi);
}

bool model_of(PyObject* o, hf_model* m, int* P) {
  if (!attr_int(o, s_kind, &m->kind) || !attr_int(o, s_n_gauss, &m->n_gauss) ||
      !attr_int(o, s_poly_degree, &m->poly_degree) || !attr_int(o, s_bin_average, &m->bin_average) ||
      !attr_double(o, s_t_shift, &m->t_shift) || !attr_double(o, s_t_scale, &m->t_scale))
    return false;
  *P = api.nparams(m);
  return *P > 0;
}

int counts_code(const at::Tensor& t) {
  switch (t.scalar_type()) {
    case c10::ScalarType::Int:
    case c10::ScalarType::UInt32:
      return HF_U32;
    case c10::ScalarType::Float:
      return HF_F32;
    case c10::ScalarType::Double:
      return HF_F64;
    default:
      return -1;
  }
}

const at::Tensor* counts_of(PyObject* o, int* code) {
  if (!o || !THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined()) return nullptr;
  *code = counts_code(t);
  return *code < 0 ? nullptr : plain(o, -1, t.scalar_type(), 0);
}

// The histogram's arrays stay referenced while a Hist lives.
struct Hist {
  Owned counts, weights, edges;
  const at::Tensor* c = nullptr;
  hf_hist h{};
  explicit Hist(PyObject* o)
      : counts(PyObject_GetAttr(o, s_counts)), weights(PyObject_GetAttr(o, s_weights)),
        edges(PyObject_GetAttr(o, s_edges)) {
    int code;
    if (!counts.o || !weights.o || !edges.o) return;
    const at::Tensor* t = counts_of(counts.o, &code);
    if (!t || t->dim() < 1 || t->dim() > 2 || !attr_range(o, s_xrange, &h.xlo, &h.xhi) ||
        !attr_range(o, s_yrange, &h.ylo, &h.yhi))
      return;
    h.counts = t->data_ptr();
    h.counts_dtype = code;
    h.nx = t->size(-1);
    h.ny = t->dim() == 2 ? t->size(0) : 1;
    const int dev = t->get_device();
    if (!is_none(weights.o)) {
      const at::Tensor* w = plain(weights.o, dev, c10::ScalarType::Float, 0);
      if (!w || w->numel() != t->numel()) return;
      h.weights = w->data_ptr<float>();
    }
    if (!is_none(edges.o)) {
      const at::Tensor* e = plain(edges.o, dev, c10::ScalarType::Double, 0);
      if (!e || t->dim() != 1 || e->numel() != t->numel() + 1) return;
      h.x_edges = e->data_ptr<double>();
    }
    c = t;
  }
};

// The current stream of the device and its context, null where context() in the
// Python code has something to do (no context yet, spares to make up).
hf_ctx* context_of(int dev, hf_stream_t* stream) {
  const hipStream_t s = c10::hip::getCurrentHIPStream(static_cast<c10::DeviceIndex>(dev)).stream();
  *stream = reinterpret_cast<hf_stream_t>(s);
  // the key's objects, kept while calls stay on one stream
  static struct {
    int dev = -1;
    hipStream_t s = nullptr;
    PyObject* key = nullptr;
  } last;
  if (last.dev != dev || last.s != s || !last.key) {
    PyObject* k = Py_BuildValue("iN", dev, PyLong_FromVoidPtr(s));
    if (!k) return nullptr;
    Py_XSETREF(last.key, k);
    last.dev = dev;
    last.s = s;
  }
  PyObject* pool = PyDict_GetItemWithError(pools, PyTuple_GET_ITEM(last.key, 0));
  if (!pool || !PyList_Check(pool) || PyList_GET_SIZE(pool) < spares) return nullptr;
  PyObject* c = PyDict_GetItemWithError(contexts, last.key);
  Owned value(c ? PyObject_GetAttr(c, s_value) : nullptr);  // of a ctypes.c_void_p
  return value.o && PyLong_Check(value.o) ? static_cast<hf_ctx*>(PyLong_AsVoidPtr(value.o)) : nullptr;
}

// The interpreter lock given up while this lives.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  Unlocked() = default;
  ~Unlocked() { PyEval_RestoreThread(state); }
  Unlocked(const Unlocked&) = delete;
  Unlocked& operator=(const Unlocked&) = delete;
};

// One call of a function here: what fails before the library is called is left
// to the Python code, what fails from then on is raised.
struct Call {
  bool made = false;
  // Runs f, a call of the library, without the interpreter lock.
  template <class F>
  bool run(hf_ctx* ctx, F&& f) {
    int rc;
    {
      Unlocked u;
      made = true;
      rc = f();
    }
    if (rc != 0) PyErr_Format(error_type, "histfit error %d: %s", rc, api.last_error(ctx));
    return rc == 0;
  }
};

// Wraps a function body: None (nothing done) where it gives no result or throws
// before the library's call.
template <class F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F&& body) {
  PyObject* r = nullptr;
  Call call;
  if (n == want && api.nparams) {
    try {
      if (!modes_active()) r = body(call);
    } catch (const std::exception& e) {
      r = nullptr;
      if (call.made) PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
      r = nullptr;
      if (call.made) PyErr_SetString(PyExc_RuntimeError, "unknown error");
    }
  }
  if (r || call.made) return r;
  PyErr_Clear();
  Py_RETURN_NONE;
}

PyObject* pack(PyObject* a, PyObject* b) {
  if (!a || !b) {
    Py_XDECREF(a);
    Py_XDECREF(b);
    return nullptr;
  }
  PyObject* r = PyTuple_Pack(2, a, b);
  Py_DECREF(a);
  Py_DECREF(b);
  return r;
}

// status: None, or i32 on the device
bool status_of(PyObject* o, int dev, int32_t** p) {
  *p = nullptr;
  if (is_none(o)) return true;
  const at::Tensor* t = plain(o, dev, c10::ScalarType::Int, 1);
  if (t) *p = t->data_ptr<int32_t>();
  return t != nullptr;
}

const at::Tensor* theta_of(PyObject* o, int dev, int P) {
  const at::Tensor* t = plain(o, dev, c10::ScalarType::Double, P);
  return t && t->numel() == P ? t : nullptr;
}

// (hist, model, theta, objective, precision, out, status)
PyObject* fast_eval(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&](Call& call) -> PyObject* {
    Hist h(a[0]);
    hf_model m{};
    int P;
    long obj, prec;
    hf_stream_t stream;
    int32_t* st;
    if (!h.c || !model_of(a[1], &m, &P) || !to_int(a[3], &obj) || !to_int(a[4], &prec)) return nullptr;
    const int dev = h.c->get_device();
    hf_ctx* ctx = context_of(dev, &stream);
    const at::Tensor* th = theta_of(a[2], dev, P);
    Out out;
    if (!ctx || !th || !status_of(a[6], dev, &st) || !out.take(a[5], *h.c, c10::ScalarType::Double, {1}))
      return nullptr;
    if (!call.run(ctx, [&] {
          return api.eval(ctx, &h.h, &m, static_cast<int32_t>(obj), static_cast<int32_t>(prec),
                          static_cast<const double*>(th->data_ptr()), static_cast<double*>(out.ptr), st,
                          stream);
        }))
      return nullptr;
    return out.wrap();
  });
}

// (hist, model, theta, objective, precision, seed, want_grad_w, free_mask, nll_out, grad_out,
//  grad_w_out, status)
PyObject* fast_grad(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&](Call& call) -> PyObject* {
    Hist h(a[0]);
    hf_model m{};
    int P;
    long obj, prec, mask;
    hf_stream_t stream;
    int32_t* st;
    if (!h.c || !model_of(a[1], &m, &P) || !to_int(a[3], &obj) || !to_int(a[4], &prec) ||
        !to_int(a[7], &mask) || mask < 0 || mask > 0xffffffffL || !PyBool_Check(a[6]))
      return nullptr;
    const int dev = h.c->get_device();
    hf_ctx* ctx = context_of(dev, &stream);
    const at::Tensor* th = theta_of(a[2], dev, P);
    const double* seed = nullptr;
    if (!is_none(a[5])) {
      const at::Tensor* s = theta_of(a[5], dev, 1);
      if (!s) return nullptr;
      seed = s->data_ptr<double>();
    }
    Out nll, grad, gw;
    if (!ctx || !th || !status_of(a[11], dev, &st)) return nullptr;
    if (!is_none(a[10]) && (!THPVariable_CheckExact(a[10]) ||
                            THPVariable_Unpack(a[10]).numel() != h.c->numel()))
      return nullptr;
    const bool want = a[6] == Py_True || !is_none(a[10]);
    if (!nll.take(a[8], *h.c, c10::ScalarType::Double, {1}) ||
        !grad.take(a[9], *h.c, c10::ScalarType::Double, {P}) ||
        (want && !gw.take(a[10], *h.c, c10::ScalarType::Float, h.c->sizes())))
      return nullptr;
    if (!call.run(ctx, [&] {
          return api.grad(ctx, &h.h, &m, static_cast<int32_t>(obj), static_cast<int32_t>(prec),
                          static_cast<const double*>(th->data_ptr()), seed, static_cast<double*>(nll.ptr),
                          static_cast<double*>(grad.ptr), static_cast<float*>(gw.ptr),
                          static_cast<uint32_t>(mask), st, stream);
        }))
      return nullptr;
    Owned x(nll.wrap()), y(grad.wrap());
    Owned z(want ? gw.wrap() : (Py_INCREF(Py_None), Py_None));
    return x.o && y.o && z.o ? PyTuple_Pack(3, x.o, y.o, z.o) : nullptr;
  });
}

// (hist, model, theta, objective, out, status)
PyObject* fast_fisher(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&](Call& call) -> PyObject* {
    Hist h(a[0]);
    hf_model m{};
    int P;
    long obj;
    hf_stream_t stream;
    int32_t* st;
    if (!h.c || !model_of(a[1], &m, &P) || !to_int(a[3], &obj)) return nullptr;
    const int dev = h.c->get_device();
    hf_ctx* ctx = context_of(dev, &stream);
    const at::Tensor* th = theta_of(a[2], dev, P);
    Out out;
    if (!ctx || !th || !status_of(a[5], dev, &st) ||
        !out.take(a[4], *h.c, c10::ScalarType::Double, {P, P}) ||
        (out.given && THPVariable_Unpack(out.given).numel() != static_cast<int64_t>(P) * P))
      return nullptr;
    if (!call.run(ctx, [&] {
          return api.fisher(ctx, &h.h, &m, static_cast<int32_t>(obj),
                            static_cast<const double*>(th->data_ptr()), static_cast<double*>(out.ptr), st,
                            stream);
        }))
      return nullptr;
    return out.wrap();
  });
}

// (fisher, objective, free_mask, out, status)
PyObject* fast_covariance(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 5, [&](Call& call) -> PyObject* {
    const at::Tensor* F = plain(a[0], -1, c10::ScalarType::Double, 1);
    long obj, mask;
    hf_stream_t stream;
    if (!F || F->dim() < 2 || F->dim() > 3 || F->size(-1) != F->size(-2) || F->size(-1) > 16 ||
        !to_int(a[1], &obj) || !to_int(a[2], &mask) || mask < 0 || mask > 0xffffffffL ||
        !is_none(a[3]) || !is_none(a[4]))
      return nullptr;
    const int64_t B = F->dim() == 2 ? 1 : F->size(0);
    hf_ctx* ctx = context_of(F->get_device(), &stream);
    if (!ctx || B > INT32_MAX) return nullptr;
    Out cov, st;
    cov.take(Py_None, *F, c10::ScalarType::Double, F->sizes());
    st.take(Py_None, *F, c10::ScalarType::Int, {B});
    if (!call.run(ctx, [&] {
          return api.covariance(ctx, static_cast<int32_t>(B), static_cast<int32_t>(F->size(-1)),
                                static_cast<int32_t>(obj), static_cast<const double*>(F->data_ptr()),
                                static_cast<uint32_t>(mask), static_cast<double*>(cov.ptr),
                                static_cast<int32_t*>(st.ptr), stream);
        }))
      return nullptr;
    PyObject* x = cov.wrap();
    return pack(x, st.wrap());
  });
}

// (events, lo, hi, model, theta, weights, want_grad, nll_out, grad_out, status)
PyObject* fast_unbinned(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&](Call& call) -> PyObject* {
    const at::Tensor* ev = plain(a[0], -1, c10::ScalarType::Double, 1);
    hf_model m{};
    int P;
    double lo, hi;
    hf_stream_t stream;
    int32_t* st;
    if (!ev || ev->dim() != 1 || !to_double(a[1], &lo) || !to_double(a[2], &hi) ||
        !model_of(a[3], &m, &P) || a[6] != Py_True)
      return nullptr;
    const int dev = ev->get_device();
    hf_ctx* ctx = context_of(dev, &stream);
    const at::Tensor* th = theta_of(a[4], dev, P);
    const float* w = nullptr;
    if (!is_none(a[5])) {
      const at::Tensor* t = plain(a[5], dev, c10::ScalarType::Float, 0);
      if (!t || t->numel() != ev->numel()) return nullptr;
      w = t->data_ptr<float>();
    }
    Out nll, grad;
    if (!ctx || !th || !status_of(a[9], dev, &st) ||
        !nll.take(a[7], *ev, c10::ScalarType::Double, {1}) ||
        !grad.take(a[8], *ev, c10::ScalarType::Double, {P}))
      return nullptr;
    if (!call.run(ctx, [&] {
          return api.unbinned(ctx, static_cast<const double*>(ev->data_ptr()), w, ev->numel(), lo, hi, &m,
                              static_cast<const double*>(th->data_ptr()), static_cast<double*>(nll.ptr),
                              static_cast<double*>(grad.ptr), st, stream);
        }))
      return nullptr;
    PyObject* x = nll.wrap();
    return pack(x, grad.wrap());
  });
}

// (counts, offsets, ranges, model, theta0, objective, precision, max_iter, ls_max, fixed_iters,
//  free_mask, edm_tol, polish_edm, hessian_init, gradient, result type)
PyObject* fast_fit(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 16, [&](Call& call) -> PyObject* {
    int code, P;
    hf_model m{};
    hf_fit_opts o{};
    long obj, prec, max_iter, ls_max, mask, hinit, gradient;
    hf_stream_t stream;
    const at::Tensor* c = counts_of(a[0], &code);
    if (!c || !model_of(a[3], &m, &P) || !to_int(a[5], &obj) || !to_int(a[6], &prec) ||
        !to_int(a[7], &max_iter) || !to_int(a[8], &ls_max) || !PyBool_Check(a[9]) ||
        !to_int(a[10], &mask) || mask < 0 || mask > 0xffffffffL || !to_double(a[11], &o.edm_tol) ||
        !to_double(a[12], &o.polish_edm) || !to_int(a[13], &hinit) || !to_int(a[14], &gradient))
      return nullptr;
    const int dev = c->get_device();
    const at::Tensor* off = plain(a[1], dev, c10::ScalarType::Long, 2);
    hf_ctx* ctx = context_of(dev, &stream);
    if (!off || off->dim() != 1 || !ctx) return nullptr;
    const int64_t B = off->numel() - 1;
    const at::Tensor* rg = plain(a[2], dev, c10::ScalarType::Double, 2 * B);
    const at::Tensor* th = plain(a[4], dev, c10::ScalarType::Double, B * P);
    if (!rg || rg->numel() != 2 * B || !th || th->numel() != B * P || B > INT32_MAX ||
        max_iter != static_cast<int32_t>(max_iter) || ls_max != static_cast<int32_t>(ls_max))
      return nullptr;
    o.max_iter = static_cast<int32_t>(max_iter);
    o.ls_max = static_cast<int32_t>(ls_max);
    o.fixed_iters = a[9] == Py_True;
    o.free_mask = static_cast<uint32_t>(mask);
    o.hessian_init = static_cast<int32_t>(hinit);
    o.gradient = static_cast<int32_t>(gradient);
    Out theta, nll, st, it, ne;
    theta.take(Py_None, *c, c10::ScalarType::Double, {B, P});
    nll.take(Py_None, *c, c10::ScalarType::Double, {B});
    st.take(Py_None, *c, c10::ScalarType::Int, {B});
    it.take(Py_None, *c, c10::ScalarType::Int, {B});
    ne.take(Py_None, *c, c10::ScalarType::Int, {B});
    if (!call.run(ctx, [&] {
          return api.fit(ctx, static_cast<int32_t>(B), c->data_ptr(), code,
                         static_cast<const int64_t*>(off->data_ptr()),
                         static_cast<const double*>(rg->data_ptr()), &m, static_cast<int32_t>(obj),
                         static_cast<int32_t>(prec), static_cast<const double*>(th->data_ptr()), &o,
                         static_cast<double*>(theta.ptr), static_cast<double*>(nll.ptr),
                         static_cast<int32_t*>(st.ptr), static_cast<int32_t*>(it.ptr),
                         static_cast<int32_t*>(ne.ptr), stream);
        }))
      return nullptr;
    Owned r1(theta.wrap()), r2(nll.wrap()), r3(st.wrap()), r4(it.wrap()), r5(ne.wrap());
    if (!r1.o || !r2.o || !r3.o || !r4.o || !r5.o) return nullptr;
    return PyObject_CallFunctionObjArgs(a[15], r1.o, r2.o, r3.o, r4.o, r5.o, nullptr);
  });
}

// (handle of libhistfit.so, contexts, pools, spares, HistfitError)
PyObject* init_api(PyObject*, PyObject* args) {
  PyObject *handle, *ctx, *pool, *error;
  Py_ssize_t n;
  if (!PyArg_ParseTuple(args, "OO!O!nO", &handle, &PyDict_Type, &ctx, &PyDict_Type, &pool, &n, &error))
    return nullptr;
  void* h = PyLong_AsVoidPtr(handle);
  if (!h) return nullptr;
  Api f;
  f.nparams = reinterpret_cast<decltype(f.nparams)>(dlsym(h, "hf_model_nparams"));
  f.eval = reinterpret_cast<decltype(f.eval)>(dlsym(h, "nll_eval"));
  f.grad = reinterpret_cast<decltype(f.grad)>(dlsym(h, "nll_grad"));
  f.unbinned = reinterpret_cast<decltype(f.unbinned)>(dlsym(h, "nll_unbinned"));
  f.fisher = reinterpret_cast<decltype(f.fisher)>(dlsym(h, "hf_nll_fisher"));
  f.covariance = reinterpret_cast<decltype(f.covariance)>(dlsym(h, "hf_fisher_covariance"));
  f.fit = reinterpret_cast<decltype(f.fit)>(dlsym(h, "fit_batch"));
  f.last_error = reinterpret_cast<decltype(f.last_error)>(dlsym(h, "hf_last_error"));
  if (!f.nparams || !f.eval || !f.grad || !f.unbinned || !f.fisher || !f.covariance || !f.fit ||
      !f.last_error) {
    PyErr_SetString(PyExc_RuntimeError, "libhistfit.so lacks an entry point");
    return nullptr;
  }
  Py_INCREF(ctx);
  Py_INCREF(pool);
  Py_INCREF(error);
  Py_XSETREF(contexts, ctx);
  Py_XSETREF(pools, pool);
  Py_XSETREF(error_type, error);
  spares = n;
  api = f;
  Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"nll_eval", FAST(fast_eval), nullptr},
    {"nll_grad", FAST(fast_grad), nullptr},
    {"nll_fisher", FAST(fast_fisher), nullptr},
    {"fisher_covariance", FAST(fast_covariance), nullptr},
    {"nll_unbinned", FAST(fast_unbinned), nullptr},
    {"fit_batch", FAST(fast_fit), nullptr},
    {"init", init_api, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() {
  struct {
    PyObject** p;
    const char* s;
  } names[] = {{&s_counts, "counts"},     {&s_weights, "weights"}, {&s_edges, "edges"},
               {&s_xrange, "xrange"},     {&s_yrange, "yrange"},   {&s_kind, "kind"},
               {&s_n_gauss, "n_gauss"},   {&s_poly_degree, "poly_degree"},
               {&s_t_shift, "t_shift"},   {&s_t_scale, "t_scale"}, {&s_bin_average, "bin_average"},
               {&s_value, "value"}};
  for (auto& n : names)
    if (!(*n.p = PyUnicode_InternFromString(n.s))) return nullptr;
  return PyModule_Create(&module);
}
