// Host side of the Python entry points: argument checks, allocation of outputs and workspaces, the
// stream, and the autograd node around the two calls of the library.  No arithmetic of its own.
//
// The smallest calls are bounded by what the host does between two launches: as Python (dataclass ->
// ctypes structure, tensor checks, a torch.autograd.Function whose backward re-enters the interpreter)
// the tiny training step (B1 H2 N128 d64) took 203 us of host time for 36 us of kernels.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include "sagebwd.h"

namespace {

using at::Tensor;

// ---- what the Python side of the package provides (looked up once) --------------------------------
PyObject* g_binding = nullptr;     // the package's `binding` module: raises the exceptions of this file

struct Names {
  PyObject *B, *H, *N, *d, *causal, *k_smooth, *q_smooth, *sm_scale, *token_major, *share_quantized, *scratch_budget, *bq, *bkv,
      *Nkv, *qk_gamma_q, *qk_gamma_k, *qk_norm_eps;
} g_names;

// Raises what binding.<fn>(args) raises; always returns nullptr.
PyObject* raise_through(const char* fn, PyObject* args) {
  if (args != nullptr) {
    PyObject* f = PyObject_GetAttrString(g_binding, fn);
    PyObject* r = f != nullptr ? PyObject_CallObject(f, args) : nullptr;
    Py_XDECREF(f);
    Py_DECREF(args);
    if (r != nullptr) {
      Py_DECREF(r);
      PyErr_SetString(PyExc_RuntimeError, "sagebwd: inconsistent host checks");
    }
  }
  return nullptr;
}
PyObject* raise_status(int status, const char* where) { return raise_through("_check", Py_BuildValue("(is)", status, where)); }

// ---- SageParams -> sagebwd_params -----------------------------------------------------------------
struct Params {
  sagebwd_params c;
  int64_t nkv() const { return c.Nkv > 0 ? c.Nkv : c.N; }
  bool token_major() const { return c.layout == SAGEBWD_LAYOUT_BNHD; }
  std::array<int64_t, 4> shape(bool kv) const {
    const int64_t n = kv ? nkv() : c.N;
    return token_major() ? std::array<int64_t, 4>{c.B, n, c.H, c.d} : std::array<int64_t, 4>{c.B, c.H, n, c.d};
  }
  std::array<int64_t, 3> lse_shape() const { return {c.B, c.H, c.N}; }
};

// (the conversions of SageParams.c(): the sizes have to be integers, the other numbers go through int() and float())
PyObject* get_int(PyObject* o, PyObject* name) {
  PyObject* v = PyObject_GetAttr(o, name);
  if (v == nullptr || PyLong_CheckExact(v) || PyBool_Check(v)) return v;
  PyObject* i = PyNumber_Long(v);
  Py_DECREF(v);
  return i;
}
bool take_int32(PyObject* v, int32_t* out) {      // (takes the reference)
  if (v == nullptr) return false;
  const long long x = PyLong_AsLongLong(v);
  Py_DECREF(v);
  if (x == -1 && PyErr_Occurred()) return false;
  *out = (int32_t)x;
  return true;
}
bool read_size(PyObject* o, PyObject* name, int32_t* out) { return take_int32(PyObject_GetAttr(o, name), out); }
bool read_int(PyObject* o, PyObject* name, int32_t* out) { return take_int32(get_int(o, name), out); }
bool read_u64(PyObject* o, PyObject* name, uint64_t* out) {
  PyObject* v = get_int(o, name);
  if (v == nullptr) return false;
  *out = PyLong_AsUnsignedLongLongMask(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}
bool read_float(PyObject* o, PyObject* name, float* out) {
  PyObject* v = PyObject_GetAttr(o, name);
  if (v == nullptr) return false;
  PyObject* f = PyNumber_Float(v);
  Py_DECREF(v);
  if (f == nullptr) return false;
  *out = (float)PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return true;
}
bool read_bool(PyObject* o, PyObject* name, bool* out) {
  PyObject* v = PyObject_GetAttr(o, name);
  if (v == nullptr) return false;
  const int t = PyObject_IsTrue(v);
  Py_DECREF(v);
  *out = t > 0;
  return t >= 0;
}
// QK-norm gain: None, or a contiguous float32 GPU tensor [d]
bool read_gain(PyObject* o, PyObject* name, int32_t d, const float** out) {
  PyObject* v = PyObject_GetAttr(o, name);
  if (v == nullptr) return false;
  bool ok = true;
  *out = nullptr;
  if (v != Py_None) {
    const Tensor* t = THPVariable_Check(v) ? &THPVariable_Unpack(v) : nullptr;
    if (t != nullptr && t->scalar_type() == at::kFloat && t->dim() == 1 && t->size(0) == d && t->is_contiguous() && t->is_cuda()) {
      *out = (const float*)t->data_ptr();
    } else {
      PyErr_Format(PyExc_ValueError, "QK-norm gain: need contiguous cuda float32 (%d,)", (int)d);
      ok = false;
    }
  }
  Py_DECREF(v);
  return ok;
}

bool read_params(PyObject* o, Params& p) {
  const Names& n = g_names;
  sagebwd_params& c = p.c;
  bool ks, qs, tm, share;
  c.reserved = 0;
  if (!read_size(o, n.B, &c.B) || !read_size(o, n.H, &c.H) || !read_size(o, n.N, &c.N) || !read_size(o, n.d, &c.d) ||
      !read_int(o, n.causal, &c.causal) || !read_bool(o, n.k_smooth, &ks) || !read_bool(o, n.q_smooth, &qs) ||
      !read_float(o, n.sm_scale, &c.sm_scale) || !read_bool(o, n.token_major, &tm) || !read_bool(o, n.share_quantized, &share) ||
      !read_u64(o, n.scratch_budget, &c.scratch_budget) || !read_int(o, n.bq, &c.bq) || !read_int(o, n.bkv, &c.bkv) ||
      !read_int(o, n.Nkv, &c.Nkv) || !read_gain(o, n.qk_gamma_q, c.d, &c.qk_gamma_q) || !read_gain(o, n.qk_gamma_k, c.d, &c.qk_gamma_k))
    return false;
  c.smooth = (ks ? SAGEBWD_SMOOTH_K : 0) | (qs ? SAGEBWD_SMOOTH_Q : 0);
  c.layout = tm ? SAGEBWD_LAYOUT_BNHD : SAGEBWD_LAYOUT_BHND;
  c.flags = (share ? SAGEBWD_FLAG_SHARE_QUANTIZED : 0) | (c.qk_gamma_q != nullptr ? SAGEBWD_FLAG_QK_NORM : 0);
  c.qk_norm_eps = 0.f;
  return c.qk_gamma_q == nullptr || read_float(o, n.qk_norm_eps, &c.qk_norm_eps);
}

// ---- tensor arguments ----------------------------------------------------------------------------
bool fits(const Tensor& t, at::ScalarType dtype, at::IntArrayRef shape) {
  return t.scalar_type() == dtype && t.sizes() == shape && t.is_contiguous() && t.is_cuda();
}
// The tensor behind a Python argument if it is what the call needs; else nullptr with the exception set.
const Tensor* expect(PyObject* o, at::ScalarType dtype, at::IntArrayRef shape, const char* name) {
  if (THPVariable_Check(o)) {
    const Tensor& t = THPVariable_Unpack(o);
    if (fits(t, dtype, shape)) return &t;
  }
  PyObject* tuple = PyTuple_New((Py_ssize_t)shape.size());
  for (size_t k = 0; tuple != nullptr && k < shape.size(); k++) PyTuple_SET_ITEM(tuple, (Py_ssize_t)k, PyLong_FromLongLong(shape[k]));
  raise_through("_expect_named", Py_BuildValue("(OsNs)", o, dtype == at::kFloat ? "float32" : "bfloat16", tuple, name));
  return nullptr;
}
// The workspace argument: any tensor, numel() bytes of which are used (None: the caller allocates).
bool workspace_arg(PyObject* o, Tensor* out) {
  if (o == Py_None) return true;
  if (!THPVariable_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "workspace: need a tensor");
    return false;
  }
  *out = THPVariable_Unpack(o);
  return true;
}

hipStream_t current_stream() { return c10::hip::getCurrentHIPStream().stream(); }
// sagebwd_workspace_bytes through `out` on the device of `like`; returns its status.
int alloc_workspace(const Params& p, bool forward_only, const Tensor& like, Tensor* out) {
  size_t fwd = 0, bwd = 0;
  const int rc = sagebwd_workspace_bytes(&p.c, &fwd, &bwd);
  if (rc == SAGEBWD_OK) *out = at::empty({(int64_t)(forward_only ? fwd : bwd)}, like.options().dtype(at::kByte));
  return rc;
}

int run_fwd(const Tensor& Q, const Tensor& K, const Tensor& V, const Tensor& O, const Tensor& L, const Params& p, const Tensor& ws) {
  return sagebwd_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), (float*)L.data_ptr(), &p.c, ws.data_ptr(),
                     (size_t)ws.numel(), (void*)current_stream());
}
int run_bwd(const Tensor& Q, const Tensor& K, const Tensor& V, const Tensor& O, const Tensor& dO, const Tensor& L, const Tensor& dQ,
            const Tensor& dK, const Tensor& dV, const Params& p, const Tensor& ws) {
  return sagebwd_bwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), dO.data_ptr(), (const float*)L.data_ptr(), dQ.data_ptr(),
                     dK.data_ptr(), dV.data_ptr(), &p.c, ws.data_ptr(), (size_t)ws.numel(), (void*)current_stream());
}

bool arg_count(Py_ssize_t n, Py_ssize_t want, const char* fn) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", fn, want, n);
  return false;
}
PyObject* wrap2(const Tensor& a, const Tensor& b) { return Py_BuildValue("(NN)", THPVariable_Wrap(a), THPVariable_Wrap(b)); }

// The interpreter lock is given up from the checks to the results, as a foreign call would do: a launch can
// block when the queue is full, and the allocator may wait for the GPU.
#define WITHOUT_GIL(body)                \
  {                                      \
    pybind11::gil_scoped_release no_gil; \
    body                                 \
  }

// fwd(Q, K, V, p, workspace | None, O | None, LSE | None) -> (O, LSE)
PyObject* py_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Params p;
  if (!arg_count(n, 7, "fwd") || !read_params(a[3], p)) return nullptr;
  const auto shp = p.shape(false), kshp = p.shape(true);
  const auto lshp = p.lse_shape();
  const Tensor *Q, *K, *V;
  Tensor ws, O, L;
  if (!(Q = expect(a[0], at::kBFloat16, shp, "Q")) || !(K = expect(a[1], at::kBFloat16, kshp, "K")) ||
      !(V = expect(a[2], at::kBFloat16, kshp, "V")) || !workspace_arg(a[4], &ws))
    return nullptr;
  if (a[5] != Py_None) {
    const Tensor* t = expect(a[5], at::kBFloat16, shp, "O");
    if (t == nullptr) return nullptr;
    O = *t;
  }
  if (a[6] != Py_None) {
    const Tensor* t = expect(a[6], at::kFloat, lshp, "LSE");
    if (t == nullptr) return nullptr;
    L = *t;
  }
  int rc = SAGEBWD_OK;
  const char* where = "sagebwd_workspace_bytes";
  WITHOUT_GIL({
    if (!ws.defined()) rc = alloc_workspace(p, true, *Q, &ws);
    if (rc == SAGEBWD_OK) {
      where = "sagebwd_fwd";
      if (!O.defined()) O = at::empty(shp, Q->options());
      if (!L.defined()) L = at::empty(lshp, Q->options().dtype(at::kFloat));
      rc = run_fwd(*Q, *K, *V, O, L, p, ws);
    }
  })
  if (rc != SAGEBWD_OK) return raise_status(rc, where);
  return wrap2(O, L);
  END_HANDLE_TH_ERRORS
}

// fwd_static(Q, K, V, p, O, LSE) -> (O, LSE)
PyObject* py_fwd_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Params p;
  if (!arg_count(n, 6, "fwd_static") || !read_params(a[3], p)) return nullptr;
  const auto shp = p.shape(false), kshp = p.shape(true);
  const auto lshp = p.lse_shape();
  const Tensor *Q, *K, *V, *O, *L;
  if (!(Q = expect(a[0], at::kBFloat16, shp, "Q")) || !(O = expect(a[4], at::kBFloat16, shp, "O")) ||
      !(K = expect(a[1], at::kBFloat16, kshp, "K")) || !(V = expect(a[2], at::kBFloat16, kshp, "V")) ||
      !(L = expect(a[5], at::kFloat, lshp, "LSE")))
    return nullptr;
  int rc;
  WITHOUT_GIL({
    rc = sagebwd_fwd_static(Q->data_ptr(), K->data_ptr(), V->data_ptr(), O->data_ptr(), (float*)L->data_ptr(), &p.c,
                            (void*)current_stream());
  })
  if (rc != SAGEBWD_OK) return raise_status(rc, "sagebwd_fwd_static");
  return wrap2(*O, *L);
  END_HANDLE_TH_ERRORS
}

// bwd(Q, K, V, O, dO, LSE, p, workspace | None, dQ | None, dK | None, dV | None) -> (dQ, dK, dV)
PyObject* py_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Params p;
  if (!arg_count(n, 11, "bwd") || !read_params(a[6], p)) return nullptr;
  const auto shp = p.shape(false), kshp = p.shape(true);
  const Tensor *Q, *K, *V, *O, *dO, *L;
  Tensor ws, grad[3];
  if (!(Q = expect(a[0], at::kBFloat16, shp, "Q")) || !(O = expect(a[3], at::kBFloat16, shp, "O")) ||
      !(dO = expect(a[4], at::kBFloat16, shp, "dO")) || !(K = expect(a[1], at::kBFloat16, kshp, "K")) ||
      !(V = expect(a[2], at::kBFloat16, kshp, "V")) || !(L = expect(a[5], at::kFloat, p.lse_shape(), "LSE")) || !workspace_arg(a[7], &ws))
    return nullptr;
  const char* names[3] = {"dQ", "dK", "dV"};
  for (int k = 0; k < 3; k++) {
    if (a[8 + k] == Py_None) continue;
    const Tensor* t = expect(a[8 + k], at::kBFloat16, k == 0 ? shp : kshp, names[k]);
    if (t == nullptr) return nullptr;
    grad[k] = *t;
  }
  int rc = SAGEBWD_OK;
  const char* where = "sagebwd_workspace_bytes";
  WITHOUT_GIL({
    if (!ws.defined()) rc = alloc_workspace(p, false, *Q, &ws);
    if (rc == SAGEBWD_OK) {
      where = "sagebwd_bwd";
      for (int k = 0; k < 3; k++)
        if (!grad[k].defined()) grad[k] = at::empty(k == 0 ? shp : kshp, Q->options());
      rc = run_bwd(*Q, *K, *V, *O, *dO, *L, grad[0], grad[1], grad[2], p, ws);
    }
  })
  if (rc != SAGEBWD_OK) return raise_status(rc, where);
  return Py_BuildValue("(NNN)", THPVariable_Wrap(grad[0]), THPVariable_Wrap(grad[1]), THPVariable_Wrap(grad[2]));
  END_HANDLE_TH_ERRORS
}

// ---- autograd --------------------------------------------------------------------------------------
// Throws the Python exception that the library's status stands for (the engine's threads hold no interpreter lock).
[[noreturn]] void throw_python(const std::function<void()>& raise) {
  pybind11::gil_scoped_acquire gil;
  raise();
  python_error err;
  err.persist();
  throw err;
}

struct SageAttentionBackward : torch::autograd::Node {
  torch::autograd::SavedVariable Q, K, V, O, L;
  Params p;
  Tensor ws;       // the forward's workspace where the backward takes psi(Q), psi(K) from it
  std::string name() const override { return "SageAttentionBackward"; }
  void release_variables() override {
    std::lock_guard<std::mutex> lock(mutex_);
    Q.reset_data(); K.reset_data(); V.reset_data(); O.reset_data(); L.reset_data();
    ws.reset();
  }
  torch::autograd::variable_list apply(torch::autograd::variable_list&& grads) override {
    std::lock_guard<std::mutex> lock(mutex_);
    at::NoGradGuard no_grad;
    const Tensor q = Q.unpack(), k = K.unpack(), v = V.unpack(), o = O.unpack(shared_from_this()), l = L.unpack();
    Tensor dO = grads[0].defined() ? grads[0].contiguous() : at::zeros_like(o);
    if (!fits(dO, at::kBFloat16, q.sizes()))
      throw_python([&] {
        THPObjectPtr t(THPVariable_Wrap(dO));
        expect(t.get(), at::kBFloat16, q.sizes(), "dO");
      });
    Params pb = p;
    Tensor w = ws;
    ws.reset();    // (a second backward through a retained graph forms psi(Q), psi(K) again: the same bits)
    int rc = SAGEBWD_OK;
    if (!w.defined()) {
      pb.c.flags &= ~SAGEBWD_FLAG_SHARE_QUANTIZED;
      rc = alloc_workspace(pb, false, q, &w);
    }
    Tensor dQ, dK, dV;
    if (rc == SAGEBWD_OK) {
      dQ = at::empty_like(q); dK = at::empty_like(k); dV = at::empty_like(v);
      rc = run_bwd(q, k, v, o, dO, l, dQ, dK, dV, pb, w);
    }
    if (rc != SAGEBWD_OK) throw_python([&] { raise_status(rc, "sagebwd_bwd"); });
    return {dQ, dK, dV};
  }
};

// A tensor whose data alone is not what the caller asked about: a dual tensor of forward-mode AD (its tangent would be
// dropped, which reads as a zero derivative), or one wrapped by a torch.func transform.
bool is_transformed(const Tensor& t) {
  constexpr c10::DispatchKeySet wrappers({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::BatchedNestedTensor,
                                          c10::DispatchKey::FuncTorchGradWrapper});
  return torch::autograd::isFwGradDefined(t) || t.key_set().has_any(wrappers);
}

// attention(Q, K, V, causal, k_smooth, q_smooth, sm_scale, token_major, share_quantized) -> (O, LSE)
PyObject* py_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (!arg_count(n, 9, "attention")) return nullptr;
  for (int k = 0; k < 3; k++) {
    if (!THPVariable_Check(a[k])) {
      PyErr_SetString(PyExc_TypeError, "sage_attention: Q, K, V are tensors");
      return nullptr;
    }
    if (is_transformed(THPVariable_Unpack(a[k]))) {
      PyErr_SetString(PyExc_NotImplementedError,
                      "sage_attention has no forward-mode derivative and no rule for torch.func transforms (vmap, grad, jvp, ...)");
      return nullptr;
    }
  }
  int flag[4];
  const int at_arg[4] = {4, 5, 7, 8};
  for (int k = 0; k < 4; k++)
    if ((flag[k] = PyObject_IsTrue(a[at_arg[k]])) < 0) return nullptr;
  const bool ks = flag[0], qs = flag[1], tm = flag[2], share = flag[3];
  int32_t causal;
  if (!take_int32(PyNumber_Long(a[3]), &causal)) return nullptr;
  THPObjectPtr scale(PyNumber_Float(a[6]));
  if (!scale) return nullptr;
  const double sm_scale = PyFloat_AS_DOUBLE(scale.get());
  const Tensor inQ = THPVariable_Unpack(a[0]), inK = THPVariable_Unpack(a[1]), inV = THPVariable_Unpack(a[2]);
  if (inQ.dim() != 4 || inK.dim() != 4) {
    PyErr_SetString(PyExc_ValueError, "sage_attention: Q, K, V need four dimensions");
    return nullptr;
  }
  Params p;
  memset(&p.c, 0, sizeof(p.c));
  p.c.B = (int32_t)inQ.size(0);
  p.c.H = (int32_t)inQ.size(tm ? 2 : 1);
  p.c.N = (int32_t)inQ.size(tm ? 1 : 2);
  p.c.d = (int32_t)inQ.size(3);
  const int32_t nkv = (int32_t)inK.size(tm ? 1 : 2);
  p.c.Nkv = nkv == p.c.N ? 0 : nkv;
  p.c.causal = causal;
  p.c.smooth = (ks ? SAGEBWD_SMOOTH_K : 0) | (qs ? SAGEBWD_SMOOTH_Q : 0);
  p.c.sm_scale = (float)sm_scale;
  p.c.layout = tm ? SAGEBWD_LAYOUT_BNHD : SAGEBWD_LAYOUT_BHND;
  p.c.flags = share ? SAGEBWD_FLAG_SHARE_QUANTIZED : 0;
  const bool track = at::GradMode::is_enabled() && (inQ.requires_grad() || inK.requires_grad() || inV.requires_grad());
  Tensor O, L;
  int rc;
  const char* where = "sagebwd_workspace_bytes";
  {
    at::NoGradGuard no_grad;
    const Tensor Q = inQ.contiguous(), K = inK.contiguous(), V = inV.contiguous();
    const auto shp = p.shape(false), kshp = p.shape(true);
    const Tensor* ts[3] = {&Q, &K, &V};
    const char* names[3] = {"Q", "K", "V"};
    for (int k = 0; k < 3; k++) {
      if (fits(*ts[k], at::kBFloat16, k == 0 ? shp : kshp)) continue;
      THPObjectPtr t(THPVariable_Wrap(*ts[k]));
      if (t) expect(t.get(), at::kBFloat16, k == 0 ? shp : kshp, names[k]);
      return nullptr;
    }
    Tensor ws;
    WITHOUT_GIL({
      // with `share` the backward takes psi(Q), psi(K) from this forward's workspace, which then has to
      // live (untouched) until the backward has run; otherwise the forward's workspace ends here
      rc = alloc_workspace(p, !share, Q, &ws);
      if (rc == SAGEBWD_OK) {
        where = "sagebwd_fwd";
        O = at::empty(shp, Q.options());
        L = at::empty(p.lse_shape(), Q.options().dtype(at::kFloat));
        rc = run_fwd(Q, K, V, O, L, p, ws);
      }
    })
    if (rc != SAGEBWD_OK) return raise_status(rc, where);
    if (track) {
      std::shared_ptr<SageAttentionBackward> node(new SageAttentionBackward(), torch::autograd::deleteNode);
      node->set_next_edges(torch::autograd::collect_next_edges(inQ, inK, inV));
      node->Q = torch::autograd::SavedVariable(Q, false);
      node->K = torch::autograd::SavedVariable(K, false);
      node->V = torch::autograd::SavedVariable(V, false);
      node->L = torch::autograd::SavedVariable(L, false);
      node->p = p;
      if (share) node->ws = ws;
      torch::autograd::set_history(O, node);
      node->O = torch::autograd::SavedVariable(O, true);
    }
  }
  return wrap2(O, L);
  END_HANDLE_TH_ERRORS
}

PyMethodDef g_methods[] = {
    {"fwd", (PyCFunction)(void (*)(void))py_fwd, METH_FASTCALL, nullptr},
    {"fwd_static", (PyCFunction)(void (*)(void))py_fwd_static, METH_FASTCALL, nullptr},
    {"bwd", (PyCFunction)(void (*)(void))py_bwd, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void (*)(void))py_attention, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_sage_host", "Host side of the SageBwd entry points", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sage_host() {
  g_binding = PyImport_ImportModule("paper_2603_02170_amd.binding");
  if (g_binding == nullptr) return nullptr;
  Names& n = g_names;
  struct { PyObject** to; const char* name; } const all[] = {
      {&n.B, "B"}, {&n.H, "H"}, {&n.N, "N"}, {&n.d, "d"}, {&n.causal, "causal"}, {&n.k_smooth, "k_smooth"}, {&n.q_smooth, "q_smooth"},
      {&n.sm_scale, "sm_scale"}, {&n.token_major, "token_major"}, {&n.share_quantized, "share_quantized"},
      {&n.scratch_budget, "scratch_budget"}, {&n.bq, "bq"}, {&n.bkv, "bkv"}, {&n.Nkv, "Nkv"}, {&n.qk_gamma_q, "qk_gamma_q"},
      {&n.qk_gamma_k, "qk_gamma_k"}, {&n.qk_norm_eps, "qk_norm_eps"}};
  for (const auto& e : all)
    if ((*e.to = PyUnicode_InternFromString(e.name)) == nullptr) return nullptr;
  return PyModule_Create(&g_module);
}
