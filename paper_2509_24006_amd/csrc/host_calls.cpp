// The host part of the calls a layer makes per pass (mask, forward, the two in one, backward) as a CPython
// module: sizes, checks of the tensors, allocation of what the caller did not pass, and the call of
// the C ABI.  A small layer is bound by this part, not by its kernels (one training step
// of 2 heads x 1110 tokens, d = 128: 191 -> 126 us, of 2 x 1024 floats, d = 64, 186 -> 109; mask and forward
// of 3 x 902, d = 64, 44 -> 28).
//
// The module decides nothing by itself.  Whatever it does not know exactly -- a tensor subclass, a
// tensor that does not fit the parameters, parameters the library refuses -- it hands back (None), and
// binding.py goes through its own checks and raises what it always raised.  An error code of the
// library comes back as an integer.  Nothing is kept between calls.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>

#include "../../include/sla.h"

namespace {

PyObject *g_device = nullptr, *g_stream = nullptr;   // torch's accessors of the current device and its raw stream

struct Call {
  const sla_params* p;
  sla_sizes_t z;
  at::ScalarType dt;
};

bool open_call(PyObject* addr, Call& c) {
  c.p = static_cast<const sla_params*>(PyLong_AsVoidPtr(addr));
  if (!c.p || sla_sizes(c.p, &c.z) != SLA_OK) return false;
  c.dt = c.p->dtype == SLA_F32 ? at::kFloat : at::kBFloat16;
  return true;
}

// a plain tensor (no subclass with functions of its own), or null
const at::Tensor* plain(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

// Q, K, V, O, dO, dQ, dK, dV: type, shape and memory order as the parameters state
bool dense(const at::Tensor* t, const Call& c) {
  const sla_params& p = *c.p;
  if (!t || !t->is_cuda() || t->scalar_type() != c.dt || t->dim() != 4) return false;
  const auto s = t->sizes();
  if (p.layout == SLA_BNHD) return s[0] == p.B && s[1] == p.N && s[2] == p.H && s[3] == p.d && t->is_contiguous();
  if (s[0] != p.B || s[1] != p.H || s[2] != p.N || s[3] != p.d) return false;
  if (p.layout != SLA_STRIDED) return t->is_contiguous();
  const auto st = t->strides();
  return st[0] == p.stride_b && st[1] == p.stride_h && st[2] == p.stride_n && st[3] == 1;
}
bool packed(const at::Tensor* t, at::IntArrayRef shape, at::ScalarType dt) {
  return t && t->is_cuda() && t->scalar_type() == dt && t->sizes() == shape && t->is_contiguous();
}
bool bytes(const at::Tensor* t, uint64_t need) {
  return t && t->is_cuda() && t->scalar_type() == at::kByte && t->dim() == 1 && t->is_contiguous() &&
         (uint64_t)t->numel() >= need;
}
bool mask(const at::Tensor* t, const Call& c) {
  return packed(t, {c.p->B, c.p->H, c.z.Tq, c.z.T}, at::kChar);
}

// An output or buffer of a call: the caller's, which has to fit, or a new one.
class Slot {
 public:
  explicit Slot(PyObject* o) : given_(o != Py_None ? o : nullptr), t_(given_ ? plain(given_) : nullptr) {}
  template <class Fits>
  bool ok(Fits fits) const { return !given_ || (t_ && fits(t_)); }
  template <class Make>
  void fill(Make make) {
    if (given_) return;
    own_ = make();
    t_ = &own_;
  }
  void* ptr() const { return t_->data_ptr(); }
  size_t size() const { return (size_t)t_->numel(); }
  PyObject* object() const {   // a new reference
    if (!given_) return THPVariable_Wrap(own_);
    Py_INCREF(given_);
    return given_;
  }

 private:
  PyObject* given_;
  at::Tensor own_;
  const at::Tensor* t_;
};

// Allocations and launches run without the interpreter lock, as they do when Python calls them one by one.
class NoGil {
 public:
  NoGil() : s_(PyEval_SaveThread()) {}
  ~NoGil() { PyEval_RestoreThread(s_); }
 private:
  PyThreadState* s_;
};

at::Tensor new_bytes(uint64_t n, const at::Tensor& like) {
  return at::empty({(int64_t)(n < 256 ? 256 : n)}, like.options().dtype(at::kByte).requires_grad(false));
}
at::Tensor new_like(const at::Tensor& t, const Call& c) {
  const auto o = t.options().requires_grad(false);
  return c.p->layout == SLA_STRIDED ? at::empty_strided(t.sizes(), t.strides(), o) : at::empty(t.sizes(), o);
}

bool current_stream(void** out) {
  PyObject* dev = PyObject_CallNoArgs(g_device);
  if (!dev) return false;
  PyObject* st = PyObject_CallFunctionObjArgs(g_stream, dev, nullptr);
  Py_DECREF(dev);
  if (!st) return false;
  *out = PyLong_AsVoidPtr(st);
  Py_DECREF(st);
  return !PyErr_Occurred();
}

PyObject* pack(std::initializer_list<PyObject*> items) {
  PyObject* t = PyTuple_New((Py_ssize_t)items.size());
  bool ok = t != nullptr;
  Py_ssize_t i = 0;
  for (PyObject* o : items) {
    ok = ok && o;
    if (t) PyTuple_SET_ITEM(t, i++, o);
    else Py_XDECREF(o);
  }
  if (ok) return t;
  Py_XDECREF(t);
  return nullptr;
}

// build_mask(params address, Q, K, workspace, Mc, luts) -> (Mc, luts, workspace)
PyObject* build_mask(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Call c;
  if (n != 6 || !open_call(a[0], c)) Py_RETURN_NONE;
  const at::Tensor *Q = plain(a[1]), *K = plain(a[2]);
  Slot ws(a[3]), Mc(a[4]), luts(a[5]);
  if (!dense(Q, c) || !dense(K, c) || !Mc.ok([&](auto t) { return mask(t, c); }) ||
      !luts.ok([&](auto t) { return bytes(t, c.z.luts_bytes); }) || !ws.ok([&](auto t) { return bytes(t, c.z.ws_mask_bytes); }))
    Py_RETURN_NONE;
  void* st;
  if (!current_stream(&st)) return nullptr;
  int rc;
  {
    NoGil free;
    Mc.fill([&] {
      return at::empty({c.p->B, c.p->H, c.z.Tq, c.z.T}, Q->options().dtype(at::kChar).requires_grad(false));
    });
    luts.fill([&] { return new_bytes(c.z.luts_bytes, *Q); });
    ws.fill([&] { return new_bytes(c.z.ws_mask_bytes, *Q); });
    rc = sla_build_mask(c.p, Q->data_ptr(), K->data_ptr(), (int8_t*)Mc.ptr(), luts.ptr(), ws.ptr(), ws.size(), st);
  }
  if (rc != SLA_OK) return PyLong_FromLong(rc);
  return pack({Mc.object(), luts.object(), ws.object()});
  END_HANDLE_TH_ERRORS
}

// forward(params address, Q, K, V, W, Mc, luts, O, saved, workspace, need_saved) -> (O, saved or None)
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Call c;
  if (n != 11 || !open_call(a[0], c)) Py_RETURN_NONE;
  const at::Tensor *Q = plain(a[1]), *K = plain(a[2]), *V = plain(a[3]), *W = plain(a[4]), *Mc = plain(a[5]),
                   *luts = plain(a[6]);
  Slot O(a[7]), saved(a[8]), ws(a[9]);
  if (!dense(Q, c) || !dense(K, c) || !dense(V, c) || !packed(W, {c.p->d, c.p->d}, c.dt) || !mask(Mc, c) ||
      !bytes(luts, c.z.luts_bytes) || !O.ok([&](auto t) { return dense(t, c); }) ||
      !saved.ok([&](auto t) { return bytes(t, c.z.saved_bytes); }) ||
      !ws.ok([&](auto t) { return bytes(t, c.z.ws_forward_bytes); }))
    Py_RETURN_NONE;
  const int need = PyObject_IsTrue(a[10]);
  if (need < 0) return nullptr;
  const bool save = need || a[8] != Py_None;
  void* st;
  if (!current_stream(&st)) return nullptr;
  int rc;
  {
    NoGil free;
    O.fill([&] { return new_like(*Q, c); });
    if (save) saved.fill([&] { return new_bytes(c.z.saved_bytes, *Q); });
    ws.fill([&] { return new_bytes(c.z.ws_forward_bytes, *Q); });
    rc = sla_forward(c.p, Q->data_ptr(), K->data_ptr(), V->data_ptr(), W->data_ptr(), (const int8_t*)Mc->data_ptr(),
                     luts->data_ptr(), O.ptr(), save ? saved.ptr() : nullptr, ws.ptr(), ws.size(), st);
  }
  if (rc != SLA_OK) return PyLong_FromLong(rc);
  if (!save) Py_INCREF(Py_None);
  return pack({O.object(), save ? saved.object() : Py_None});
  END_HANDLE_TH_ERRORS
}

// mask_forward(params address, Q, K, V, W, need_saved) -> (Mc, luts, O, saved or None)
PyObject* mask_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Call c;
  if (n != 6 || !open_call(a[0], c)) Py_RETURN_NONE;
  const at::Tensor *Q = plain(a[1]), *K = plain(a[2]), *V = plain(a[3]), *W = plain(a[4]);
  if (!dense(Q, c) || !dense(K, c) || !dense(V, c) || !packed(W, {c.p->d, c.p->d}, c.dt)) Py_RETURN_NONE;
  const int save = PyObject_IsTrue(a[5]);
  if (save < 0) return nullptr;
  void* st;
  if (!current_stream(&st)) return nullptr;
  at::Tensor Mc, luts, O, saved;
  int rc;
  {
    NoGil free;
    Mc = at::empty({c.p->B, c.p->H, c.z.Tq, c.z.T}, Q->options().dtype(at::kChar).requires_grad(false));
    luts = new_bytes(c.z.luts_bytes, *Q);
    O = new_like(*Q, c);
    if (save) saved = new_bytes(c.z.saved_bytes, *Q);
    const at::Tensor wm = new_bytes(c.z.ws_mask_bytes, *Q), wf = new_bytes(c.z.ws_forward_bytes, *Q);
    rc = sla_mask_forward(c.p, Q->data_ptr(), K->data_ptr(), V->data_ptr(), W->data_ptr(), (int8_t*)Mc.data_ptr(),
                          luts.data_ptr(), wm.data_ptr(), (size_t)wm.numel(), O.data_ptr(), save ? saved.data_ptr() : nullptr,
                          wf.data_ptr(), (size_t)wf.numel(), st);
  }
  if (rc != SLA_OK) return PyLong_FromLong(rc);
  if (!save) Py_INCREF(Py_None);
  return pack({THPVariable_Wrap(Mc), THPVariable_Wrap(luts), THPVariable_Wrap(O), save ? THPVariable_Wrap(saved) : Py_None});
  END_HANDLE_TH_ERRORS
}

// backward(params address, Q, K, V, W, Mc, luts, saved, dO, workspace, dQ, dK, dV, dW, dW in bf16) -> (dQ, dK, dV, dW)
PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Call c;
  if (n != 15 || !open_call(a[0], c)) Py_RETURN_NONE;
  const at::Tensor *Q = plain(a[1]), *K = plain(a[2]), *V = plain(a[3]), *W = plain(a[4]), *Mc = plain(a[5]),
                   *luts = plain(a[6]), *saved = plain(a[7]), *dO = plain(a[8]);
  Slot ws(a[9]), dQ(a[10]), dK(a[11]), dV(a[12]), dW(a[13]);
  const int w16 = PyObject_IsTrue(a[14]);
  if (w16 < 0) return nullptr;
  const at::ScalarType wt = w16 ? at::kBFloat16 : at::kFloat;
  const auto fits = [&](auto t) { return dense(t, c); };
  if (!dense(Q, c) || !dense(K, c) || !dense(V, c) || !dense(dO, c) || !packed(W, {c.p->d, c.p->d}, c.dt) ||
      !mask(Mc, c) || !bytes(luts, c.z.luts_bytes) || !bytes(saved, c.z.saved_bytes) || !dQ.ok(fits) || !dK.ok(fits) ||
      !dV.ok(fits) || !dW.ok([&](auto t) { return packed(t, {c.p->d, c.p->d}, wt); }) ||
      !ws.ok([&](auto t) { return bytes(t, c.z.ws_backward_bytes); }))
    Py_RETURN_NONE;
  void* st;
  if (!current_stream(&st)) return nullptr;
  int rc;
  {
    NoGil free;
    dQ.fill([&] { return new_like(*Q, c); });
    dK.fill([&] { return new_like(*K, c); });
    dV.fill([&] { return new_like(*V, c); });
    dW.fill([&] { return at::empty({c.p->d, c.p->d}, Q->options().dtype(wt).requires_grad(false)); });
    ws.fill([&] { return new_bytes(c.z.ws_backward_bytes, *Q); });
    rc = sla_backward_typed(c.p, Q->data_ptr(), K->data_ptr(), V->data_ptr(), W->data_ptr(),
                            (const int8_t*)Mc->data_ptr(), luts->data_ptr(), saved->data_ptr(), dO->data_ptr(),
                            dQ.ptr(), dK.ptr(), dV.ptr(), dW.ptr(), w16 ? SLA_BF16 : SLA_F32, ws.ptr(), ws.size(), st);
  }
  if (rc != SLA_OK) return PyLong_FromLong(rc);
  return pack({dQ.object(), dK.object(), dV.object(), dW.object()});
  END_HANDLE_TH_ERRORS
}

PyMethodDef g_methods[] = {
    {"build_mask", (PyCFunction)(void (*)(void))build_mask, METH_FASTCALL, nullptr},
    {"forward", (PyCFunction)(void (*)(void))forward, METH_FASTCALL, nullptr},
    {"mask_forward", (PyCFunction)(void (*)(void))mask_forward, METH_FASTCALL, nullptr},
    {"backward", (PyCFunction)(void (*)(void))backward, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_sla_host", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sla_host(void) {
  PyObject* tc = PyImport_ImportModule("torch._C");
  if (!tc) return nullptr;
  g_device = PyObject_GetAttrString(tc, "_cuda_getDevice");
  g_stream = g_device ? PyObject_GetAttrString(tc, "_cuda_getCurrentRawStream") : nullptr;
  Py_DECREF(tc);
  return g_stream ? PyModule_Create(&g_module) : nullptr;
}
