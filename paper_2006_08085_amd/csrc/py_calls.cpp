// The Python calls of the hot path in native code: argument checks and the call of the C entry point, nothing else.
//
// A small step is a few microseconds on the GPU; checking four tensors and marshalling ten arguments in Python takes as long.
// A Calls object belongs to one Context.  Each method takes what the Context method of its name takes, checks it the same way
// and returns the status of the entry point, or None without having called it if anything is not of the plain kind (another
// tensor class, a number that is not a float or an int, a check that fails): the Context then goes through ctypes, which
// accepts more kinds and words the refusals.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <new>

#include "detag.h"

namespace {

struct Entries {
  decltype(&detag_gossip_accel) gossip_accel;
  decltype(&detag_track) track;
  decltype(&detag_step) step;
  decltype(&detag_dpsgd_step) dpsgd_step;
  decltype(&detag_gossip_round) gossip_round;
  decltype(&detag_gossip_rounds) gossip_rounds;
  decltype(&detag_accumulate) accumulate;
  decltype(&detag_phase_end) phase_end;
  decltype(&detag_defacto_update) defacto_update;
  decltype(&detag_grad_quadratic_diag) grad_quadratic_diag;
  decltype(&detag_step_quadratic) step_quadratic;
  decltype(&detag_grad_lstsq) grad_lstsq;
  decltype(&detag_grad_softmax_bf16) grad_softmax_bf16;
  decltype(&detag_mean) mean;
  decltype(&detag_consensus_error) consensus_error;
  decltype(&detag_average_consensus) average_consensus;
} g_entry;
PyObject *g_current_device, *g_current_stream;  // torch's, without building the Stream object around the handle

struct Calls {
  PyObject_HEAD
  detag_ctx *ctx;
  int64_t n, d, ld;
  bool bf16;
};

// Arguments in turn; `ok` turns false at the first that is not plain.
struct Args {
  const Calls *c;
  PyObject *const *a;
  bool ok;

  const at::Tensor *tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return ok = false, nullptr;
    return &THPVariable_Unpack(o);
  }
  void *matrix(at::ScalarType type) {  // an n x ld row-major GPU matrix
    if (!ok) return nullptr;
    const at::Tensor *t = tensor(*a++);
    if (!t) return nullptr;
    ok = t->is_cuda() && t->scalar_type() == type && t->dim() == 2 && t->stride(0) == c->ld && t->stride(1) == 1 &&
         t->size(0) == c->n && t->size(1) >= c->d;
    return ok ? t->data_ptr() : nullptr;
  }
  void *state() { return matrix(c->bf16 ? at::kBFloat16 : at::kFloat); }
  float *f32() { return static_cast<float *>(matrix(at::kFloat)); }
  template <class F>
  float *plain(F &&fits) {  // a contiguous float32 GPU tensor that fits(t)
    if (!ok) return nullptr;
    const at::Tensor *t = tensor(*a++);
    if (!t) return nullptr;
    ok = t->is_cuda() && t->scalar_type() == at::kFloat && t->is_contiguous() && fits(*t);
    return ok ? static_cast<float *>(t->data_ptr()) : nullptr;
  }
  float *curvature(int32_t *per_worker, bool vector_only) {  // a vector of length >= d, or one row per worker
    if (!ok) return nullptr;
    const at::Tensor *t = tensor(*a);
    if (!t) return nullptr;
    *per_worker = t->dim() == 2;
    if (*per_worker) return f32();
    return plain([&](const at::Tensor &h) { return (!vector_only || h.dim() == 1) && h.numel() >= c->d; });
  }
  double real() {
    PyObject *o = *a++;
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    if (!PyLong_CheckExact(o)) return ok = false, 0.0;
    const double v = PyLong_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) PyErr_Clear(), ok = false;
    return v;
  }
  uint64_t integer() {  // wraps like a ctypes integer
    PyObject *o = *a++;
    if (!PyLong_CheckExact(o)) return ok = false, 0;
    const uint64_t v = PyLong_AsUnsignedLongLongMask(o);
    if (v == uint64_t(-1) && PyErr_Occurred()) PyErr_Clear(), ok = false;
    return v;
  }
  void *stream() {  // None: the current one
    if (!ok) return nullptr;
    return *a == Py_None ? current_stream() : reinterpret_cast<void *>(integer());
  }
  void *current_stream() {
    if (!ok) return nullptr;
    PyObject *dev = PyObject_CallNoArgs(g_current_device);
    PyObject *s = dev ? PyObject_CallOneArg(g_current_stream, dev) : nullptr;
    void *p = s ? PyLong_AsVoidPtr(s) : nullptr;
    Py_XDECREF(dev);
    Py_XDECREF(s);
    if (PyErr_Occurred()) PyErr_Clear(), ok = false;
    return p;
  }
};

struct WithoutInterpreter {  // other Python threads run; held again when this goes, however that comes about
  PyThreadState *state = PyEval_SaveThread();
  ~WithoutInterpreter() { PyEval_RestoreThread(state); }
};

// body(args) reads the arguments and returns the call as a function of nothing.
template <class F>
PyObject *call(PyObject *self, PyObject *const *a, Py_ssize_t nargs, Py_ssize_t want, F &&body) {
  const Calls *c = reinterpret_cast<const Calls *>(self);
  if (!c->ctx || nargs != want) Py_RETURN_NONE;
  Args args{c, a, true};
  detag_status st = DETAG_OK;
  try {
    auto go = body(args);
    if (!args.ok) Py_RETURN_NONE;
    WithoutInterpreter released;
    st = go();
  } catch (const std::bad_alloc &) {  // the entry points should not, but not every one of them ends its exceptions
    return PyErr_NoMemory();
  } catch (...) {  // a tensor without storage: the other way words it
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  return PyLong_FromLong(st);
}

#define DETAG_METHOD(name) PyObject *name(PyObject *self, PyObject *const *a, Py_ssize_t n)

DETAG_METHOD(gossip_accel) {  // Z, K, eta, stream
  return call(self, a, n, 4, [](Args &x) {
    void *z = x.state();
    const int32_t K = int32_t(x.integer());
    const double eta = x.real();
    void *s = x.stream();
    return [=, c = x.c->ctx] { return g_entry.gossip_accel(c, z, K, eta, s); };
  });
}
DETAG_METHOD(track) {  // Y, G_new, G_old
  return call(self, a, n, 3, [](Args &x) {
    void *y = x.state();
    const float *gn = x.f32(), *go = x.f32();
    void *s = x.current_stream();
    return [=, c = x.c->ctx] { return g_entry.track(c, y, gn, go, s); };
  });
}
DETAG_METHOD(step) {  // X, Y, G_new, G_old, alpha, K, eta, variant
  return call(self, a, n, 8, [](Args &p) {
    void *x = p.state(), *y = p.state();
    const float *gn = p.f32(), *go = p.f32();
    const double alpha = p.real();
    const int32_t K = int32_t(p.integer());
    const double eta = p.real();
    const int32_t variant = int32_t(p.integer());
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.step(c, x, y, gn, go, alpha, K, eta, variant, s); };
  });
}
DETAG_METHOD(dpsgd_step) {  // X, G, alpha
  return call(self, a, n, 3, [](Args &p) {
    void *x = p.state();
    const float *g = p.f32();
    const double alpha = p.real();
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.dpsgd_step(c, x, g, alpha, s); };
  });
}
DETAG_METHOD(gossip_round) {  // Z_cur, Z_prev, Z_out, eta, stream
  return call(self, a, n, 5, [](Args &p) {
    void *cur = p.state(), *prev = p.state(), *out = p.state();
    const double eta = p.real();
    void *s = p.stream();
    return [=, c = p.c->ctx] { return g_entry.gossip_round(c, cur, prev, out, eta, s); };
  });
}
DETAG_METHOD(gossip_rounds) {  // Z, Z2, R, eta, stream
  return call(self, a, n, 5, [](Args &p) {
    void *z = p.state(), *z2 = p.state();
    const int32_t R = int32_t(p.integer());
    const double eta = p.real();
    void *s = p.stream();
    return [=, c = p.c->ctx] { return g_entry.gossip_rounds(c, z, z2, R, eta, s); };
  });
}
DETAG_METHOD(accumulate) {  // G_acc, g, scale
  return call(self, a, n, 3, [](Args &p) {
    float *acc = p.f32();
    const float *g = p.f32();
    const double scale = p.real();
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.accumulate(c, acc, g, scale, s); };
  });
}
DETAG_METHOD(phase_end) {  // X, X_tilde, Y, G_k, G_km1, alpha
  return call(self, a, n, 6, [](Args &p) {
    void *x = p.state(), *xt = p.state(), *y = p.state();
    const float *gk = p.f32();
    float *gm = p.f32();
    const double alpha = p.real();
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.phase_end(c, x, xt, y, gk, gm, alpha, s); };
  });
}
DETAG_METHOD(defacto_update) {  // X, X_tilde, G, scale
  return call(self, a, n, 4, [](Args &p) {
    void *x = p.state(), *xt = p.state();
    float *g = p.f32();
    const double scale = p.real();
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.defacto_update(c, x, xt, g, scale, s); };
  });
}
DETAG_METHOD(grad_quadratic_diag) {  // X, h, b, G, sigma, seed, step (a noise array: not here)
  return call(self, a, n, 7, [](Args &p) {
    const void *x = p.state();
    int32_t per_worker = 0;
    const float *h = p.curvature(&per_worker, false), *b = p.f32();
    float *g = p.f32();
    const float sigma = float(p.real());
    const uint64_t seed = p.integer();
    const uint32_t step = uint32_t(p.integer());
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.grad_quadratic_diag(c, x, h, per_worker, b, nullptr, sigma, seed, step, g, s); };
  });
}
DETAG_METHOD(step_quadratic) {  // X, Y, G, h, b, alpha, K, sigma, seed, step, eta, variant
  return call(self, a, n, 12, [](Args &p) {
    void *x = p.state(), *y = p.state();
    float *g = p.f32();
    int32_t per_worker = 0;
    const float *h = p.curvature(&per_worker, true), *b = p.f32();
    const double alpha = p.real();
    const int32_t K = int32_t(p.integer());
    const float sigma = float(p.real());
    const uint64_t seed = p.integer();
    const uint32_t step = uint32_t(p.integer());
    const double eta = p.real();
    const int32_t variant = int32_t(p.integer());
    void *s = p.current_stream();
    return [=, c = p.c->ctx] {
      return g_entry.step_quadratic(c, x, y, g, h, per_worker, b, sigma, seed, step, alpha, K, eta, variant, s);
    };
  });
}
DETAG_METHOD(grad_lstsq) {  // X, A, b, G
  return call(self, a, n, 4, [](Args &p) {
    const void *x = p.state();
    int64_t m = 0;
    const float *A = p.plain([&](const at::Tensor &t) {
      if (t.dim() != 3 || t.size(0) != p.c->n || t.size(2) != p.c->d) return false;
      m = t.size(1);
      return true;
    });
    const float *b = p.plain([&](const at::Tensor &t) { return t.dim() == 2 && t.size(0) == p.c->n && t.size(1) == m; });
    float *g = p.f32();
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.grad_lstsq(c, x, A, b, int32_t(m), g, s); };
  });
}

DETAG_METHOD(grad_softmax_bf16) {  // X, feats, labels, batch, C, G, loss
  return call(self, a, n, 7, [](Args &p) {
    const void *x = p.state();
    const at::Tensor *f = nullptr, *lab = nullptr, *bat = nullptr;
    if (p.ok) {
      f = p.tensor(p.a[0]), lab = p.tensor(p.a[1]), bat = p.tensor(p.a[2]);
      p.a += 3;
    }
    if (p.ok) {
      const int64_t workers = p.c->n;
      p.ok = f->is_cuda() && f->scalar_type() == at::kBFloat16 && f->is_contiguous() && f->dim() == 3 && f->size(0) == workers &&
             lab->is_cuda() && lab->scalar_type() == at::kInt && lab->is_contiguous() && lab->dim() == 2 &&
             lab->size(0) == workers && lab->size(1) == f->size(1) && bat->is_cuda() && bat->scalar_type() == at::kInt &&
             bat->is_contiguous() && bat->dim() == 2 && bat->size(0) == workers;
    }
    const int32_t S = p.ok ? int32_t(f->size(1)) : 0, F = p.ok ? int32_t(f->size(2)) : 0, B = p.ok ? int32_t(bat->size(1)) : 0;
    const auto *fp = p.ok ? static_cast<const uint16_t *>(f->data_ptr()) : nullptr;
    const auto *lp = p.ok ? static_cast<const int32_t *>(lab->data_ptr()) : nullptr;
    const auto *bp = p.ok ? static_cast<const int32_t *>(bat->data_ptr()) : nullptr;
    const int32_t C = p.ok ? int32_t(p.integer()) : 0;
    float *g = p.f32(), *loss = nullptr;
    if (p.ok && *p.a != Py_None) loss = p.plain([&](const at::Tensor &t) { return t.numel() >= p.c->n; });
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.grad_softmax_bf16(c, x, fp, lp, bp, S, F, C, B, g, loss, s); };
  });
}
DETAG_METHOD(mean) {  // X, out
  return call(self, a, n, 2, [](Args &p) {
    const void *x = p.state();
    float *out = p.plain([&](const at::Tensor &t) { return t.numel() >= p.c->d; });
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.mean(c, x, out, s); };
  });
}
DETAG_METHOD(consensus_error) {  // X, out
  return call(self, a, n, 2, [](Args &p) {
    const void *x = p.state();
    const at::Tensor *t = p.ok ? p.tensor(*p.a) : nullptr;
    if (t) p.ok = t->is_cuda() && t->scalar_type() == at::kDouble && t->numel() >= 1;
    double *out = p.ok ? static_cast<double *>(t->data_ptr()) : nullptr;
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.consensus_error(c, x, out, s); };
  });
}
DETAG_METHOD(average_consensus) {  // factors, Z
  return call(self, a, n, 2, [](Args &p) {
    const auto *f = reinterpret_cast<const detag_factors *>(p.integer());
    void *z = p.state();
    void *s = p.current_stream();
    return [=, c = p.c->ctx] { return g_entry.average_consensus(c, f, z, s); };
  });
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
constexpr PyMethodDef method(const char *name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyObject *calls_new(PyTypeObject *type, PyObject *args, PyObject *) {  // handle, n, d, ld, bf16
  unsigned long long handle;
  long long n, d, ld;
  int bf16;
  if (!PyArg_ParseTuple(args, "KLLLp", &handle, &n, &d, &ld, &bf16)) return nullptr;
  PyObject *o = type->tp_alloc(type, 0);
  if (!o) return nullptr;
  Calls *c = reinterpret_cast<Calls *>(o);
  c->ctx = reinterpret_cast<detag_ctx *>(handle), c->n = n, c->d = d, c->ld = ld, c->bf16 = bf16 != 0;
  return o;
}
PyObject *calls_close(PyObject *self, PyObject *) {  // the context is gone: nothing is called any more
  reinterpret_cast<Calls *>(self)->ctx = nullptr;
  Py_RETURN_NONE;
}

// bind({name: address of the entry point}, current device, current raw stream of a device)
PyObject *bind(PyObject *, PyObject *args) {
  PyObject *entries, *device, *stream;
  if (!PyArg_ParseTuple(args, "O!OO", &PyDict_Type, &entries, &device, &stream)) return nullptr;
  Entries e;
  auto take = [&](auto &f, const char *name) {
    PyObject *v = PyDict_GetItemString(entries, name);
    f = v ? reinterpret_cast<std::decay_t<decltype(f)>>(PyLong_AsVoidPtr(v)) : nullptr;
    if (!f && !PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "no address of %s", name);
    return f != nullptr;
  };
  if (!take(e.gossip_accel, "detag_gossip_accel") || !take(e.track, "detag_track") || !take(e.step, "detag_step") ||
      !take(e.dpsgd_step, "detag_dpsgd_step") || !take(e.gossip_round, "detag_gossip_round") ||
      !take(e.gossip_rounds, "detag_gossip_rounds") || !take(e.accumulate, "detag_accumulate") ||
      !take(e.phase_end, "detag_phase_end") || !take(e.defacto_update, "detag_defacto_update") ||
      !take(e.grad_quadratic_diag, "detag_grad_quadratic_diag") || !take(e.step_quadratic, "detag_step_quadratic") ||
      !take(e.grad_lstsq, "detag_grad_lstsq") || !take(e.grad_softmax_bf16, "detag_grad_softmax_bf16") ||
      !take(e.mean, "detag_mean") || !take(e.consensus_error, "detag_consensus_error") ||
      !take(e.average_consensus, "detag_average_consensus"))
    return nullptr;
  g_entry = e;
  Py_INCREF(device);
  Py_INCREF(stream);
  Py_XSETREF(g_current_device, device);
  Py_XSETREF(g_current_stream, stream);
  Py_RETURN_NONE;
}

PyMethodDef calls_methods[] = {method<gossip_accel>("gossip_accel"),
                               method<track>("track"),
                               method<step>("step"),
                               method<dpsgd_step>("dpsgd_step"),
                               method<gossip_round>("gossip_round"),
                               method<gossip_rounds>("gossip_rounds"),
                               method<accumulate>("accumulate"),
                               method<phase_end>("phase_end"),
                               method<defacto_update>("defacto_update"),
                               method<grad_quadratic_diag>("grad_quadratic_diag"),
                               method<step_quadratic>("step_quadratic"),
                               method<grad_lstsq>("grad_lstsq"),
                               method<grad_softmax_bf16>("grad_softmax_bf16"),
                               method<mean>("mean"),
                               method<consensus_error>("consensus_error"),
                               method<average_consensus>("average_consensus"),
                               {"close", calls_close, METH_NOARGS, nullptr},
                               {nullptr, nullptr, 0, nullptr}};
PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyMethodDef module_methods[] = {{"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, module_methods};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  calls_type.tp_name = "_calls.Calls";
  calls_type.tp_basicsize = sizeof(Calls);
  calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
  calls_type.tp_new = calls_new;
  calls_type.tp_methods = calls_methods;
  if (PyType_Ready(&calls_type) < 0) return nullptr;
  PyObject *m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  Py_INCREF(&calls_type);
  if (PyModule_AddObject(m, "Calls", reinterpret_cast<PyObject *>(&calls_type)) < 0) return Py_DECREF(m), nullptr;
  return m;
}
