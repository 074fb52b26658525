// The binding's hot path: the calls a serving or training loop makes on every request, from torch tensors to the C ABI,
// as one CPython extension.  The same steps in Python and ctypes (checks of up to fourteen tensors, output allocation, the
// workspace's size and lookup, the device guard, marshalling of some thirty arguments) took more host time than a small
// request takes on the GPU.  Host time of a whole call, launches included: lime_request 31 -> 16 us (four launches),
// lime_request_prepared 25 -> 12, lime_score_candidates_gathered 19 -> 9, lime_scores 40 -> 30.
//
// Every function takes its arguments by position (binding.py has the public signatures and defaults), checks what
// binding.py always checked, raises the same exceptions, and enqueues on `stream` or the tensors' device's current stream.
// The interpreter lock is released around the library's call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <array>
#include <initializer_list>
#include <map>
#include <utility>
#include <vector>

#include "../../../include/lime.h"

namespace {

using at::Tensor;

struct PyFailed {};  // a Python exception is set

PyObject* g_lime_error = nullptr;  // binding.LimeError

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw PyFailed{};
}

// ------------------------------------------------------------------------------------------------- arguments
class Args {
 public:
  Args(PyObject* const* args, Py_ssize_t n, Py_ssize_t want) : a_(args) {
    if (n != want) raise(PyExc_TypeError, "wrong number of arguments");
  }
  // nullptr for None: `required` where the call's sizes come from the tensor, otherwise the library says what it needs.
  const Tensor* tensor(bool required = true) {
    PyObject* o = a_[i_++];
    if (o == Py_None) {
      if (required) raise(PyExc_ValueError, "a required tensor is None");
      return nullptr;
    }
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "a torch tensor is expected");
    return &THPVariable_Unpack(o);
  }
  int32_t integer() {
    const long v = PyLong_AsLong(a_[i_++]);
    if (v == -1 && PyErr_Occurred()) throw PyFailed{};
    if (v < INT32_MIN || v > INT32_MAX) raise(PyExc_OverflowError, "an integer argument does not fit 32 bits");
    return static_cast<int32_t>(v);
  }
  float number() {
    const double v = PyFloat_AsDouble(a_[i_++]);
    if (v == -1.0 && PyErr_Occurred()) throw PyFailed{};
    return static_cast<float>(v);
  }
  bool truth() {
    const int v = PyObject_IsTrue(a_[i_++]);
    if (v < 0) throw PyFailed{};
    return v != 0;
  }
  PyObject* object() { return a_[i_++]; }

 private:
  PyObject* const* a_;
  Py_ssize_t i_ = 0;
};

void* ptr(const Tensor* t) { return t == nullptr ? nullptr : t->data_ptr(); }
const int32_t* ints(const Tensor* t) { return static_cast<const int32_t*>(ptr(t)); }

// Tensors of one call: contiguous, on the GPU, of one dtype and device; the first of them is returned.
const Tensor& check(std::initializer_list<const Tensor*> tensors) {
  const Tensor* first = nullptr;
  for (const Tensor* t : tensors) {
    if (t == nullptr) continue;
    if (first == nullptr) first = t;
    if (!t->is_cuda() || !t->is_contiguous()) raise(PyExc_ValueError, "tensors must be contiguous CUDA tensors");
    if (t->scalar_type() != first->scalar_type() || t->device() != first->device())
      raise(PyExc_ValueError, "tensors must share dtype and device");
  }
  if (first->scalar_type() != at::kFloat && first->scalar_type() != at::kBFloat16)
    raise(PyExc_TypeError, "unsupported tensor dtype: float32 or bfloat16 is expected");
  return *first;
}
int32_t dtype_code(const Tensor& t) { return t.scalar_type() == at::kBFloat16 ? LIME_BF16 : LIME_F32; }

int32_t dim(const Tensor& t, int i) { return static_cast<int32_t>(t.size(i)); }
void want_dims(const Tensor& t, int n, const char* what) {
  if (t.dim() != n) raise(PyExc_ValueError, what);
}

const Tensor* check_lens(const Tensor* lens, int32_t B) {
  if (lens != nullptr && (lens->scalar_type() != at::kInt || !lens->is_cuda() || lens->numel() != B || !lens->is_contiguous()))
    raise(PyExc_ValueError, "lens must be a contiguous CUDA int32 tensor of B entries");
  return lens;
}

struct Links {
  int32_t m;
  int64_t stride;  // 0: [m, d] shared; m d: [B, m, d] per user
};
Links links_of(const Tensor& LC, int32_t B) {
  if (LC.dim() == 2) return {dim(LC, 0), 0};
  if (LC.dim() != 3 || LC.size(0) != B) raise(PyExc_ValueError, "per-user links must be [B, m, d]");
  return {dim(LC, 1), LC.size(1) * LC.size(2)};
}

// The caller's tensor, or a new one like `like`.
struct Out {
  Tensor t;
  Out(const Tensor* given, at::IntArrayRef sizes, const Tensor& like) : t(given != nullptr ? *given : at::empty(sizes, like.options())) {}
};

// ------------------------------------------------------------------------------------------------- stream and workspace
// A grow-only scratch buffer per (device, stream), see binding.get_workspace; guarded by the interpreter lock.
std::map<std::pair<int, void*>, Tensor>& workspaces() {
  static auto* m = new std::map<std::pair<int, void*>, Tensor>();  // (never destroyed: torch may be gone by then)
  return *m;
}

void* stream_handle(PyObject* stream, int device) {
  if (stream == Py_None) return c10::hip::getCurrentHIPStream(static_cast<c10::DeviceIndex>(device)).stream();
  PyObject* h = PyObject_GetAttrString(stream, "cuda_stream");
  if (h == nullptr) throw PyFailed{};
  void* p = h == Py_None ? nullptr : PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (p == nullptr && PyErr_Occurred()) throw PyFailed{};
  return p;
}

const Tensor& shared_workspace(size_t bytes, at::Device device, void* stream) {
  static auto* outgrown = new std::vector<Tensor>();  // work already queued may still use them
  Tensor& ws = workspaces()[{device.index(), stream}];
  if (!ws.defined() || static_cast<size_t>(ws.numel()) < bytes) {
    size_t want = std::max<size_t>(bytes, 256);
    if (ws.defined()) {
      outgrown->push_back(ws);
      want = std::max<size_t>(want, 2 * ws.numel());
    }
    ws = at::empty({static_cast<int64_t>(want)}, at::TensorOptions().dtype(at::kByte).device(device));
  }
  return ws;
}

// Device guard, stream and workspace of a call; then the call itself.
class Scope {
 public:
  Scope(const Tensor& like, PyObject* stream, const Tensor* workspace, size_t need)
      : guard_(like.device()), stream_(stream_handle(stream, like.device().index())),
        ws_(workspace != nullptr ? *workspace : shared_workspace(need, like.device(), stream_)) {}
  void* ws() const { return ws_.data_ptr(); }
  size_t bytes() const { return static_cast<size_t>(ws_.numel()); }
  void* stream() const { return stream_; }

 private:
  c10::DeviceGuard guard_;
  void* stream_;
  Tensor ws_;
};

[[noreturn]] void lime_failed(int32_t status, const char* text) {
  PyObject* e = PyObject_CallFunction(g_lime_error, "is", static_cast<int>(status), text);
  if (e != nullptr) {
    PyErr_SetObject(g_lime_error, e);
    Py_DECREF(e);
  }
  throw PyFailed{};
}

// The interpreter lock given up for the lifetime of the object, taken back also when an exception passes.
class Unlocked {
 public:
  Unlocked() : state_(PyEval_SaveThread()) {}
  ~Unlocked() { PyEval_RestoreThread(state_); }
  Unlocked(const Unlocked&) = delete;
  Unlocked& operator=(const Unlocked&) = delete;

 private:
  PyThreadState* state_;
};

// One entry point of the library.  Its arguments are values: a tensor's pointer is taken at the call, under the lock, where
// a tensor that has none (vmap's and other wrappers) may raise.
template <typename... P, typename... A>
void call(int32_t (*entry_point)(P...), A... args) {
  int32_t status;
  {
    Unlocked unlocked;
    status = entry_point(args...);
  }
  if (status != LIME_OK) lime_failed(status, lime_last_error());
}

PyObject* wrap(const Tensor& t) { return THPVariable_Wrap(t); }
PyObject* pair(const Tensor& a, const Tensor* b) {
  PyObject* t = PyTuple_New(2);
  if (t == nullptr) throw PyFailed{};
  PyTuple_SET_ITEM(t, 0, wrap(a));
  if (b != nullptr) {
    PyTuple_SET_ITEM(t, 1, wrap(*b));
  } else {
    Py_INCREF(Py_None);
    PyTuple_SET_ITEM(t, 1, Py_None);
  }
  return t;
}

// ------------------------------------------------------------------------------------------------- the calls
// (E, lens, LC, Wq, Wk, Wv, h, scale, LP, OS, want_os, xor, workspace, stream) -> (LP, OS or None)
PyObject* history(Args a) {
  const Tensor *E = a.tensor(), *lens = a.tensor(false), *LC = a.tensor(), *Wq = a.tensor(false), *Wk = a.tensor(false), *Wv = a.tensor(false);
  const int32_t h = a.integer();
  const float scale = a.number();
  const Tensor *LPin = a.tensor(false), *OSin = a.tensor(false);
  const bool want_os = a.truth(), is_xor = a.truth();
  const Tensor* workspace = a.tensor(false);
  const Tensor& like = check({E, LC, Wq, Wk, Wv, LPin, OSin});
  want_dims(*E, 3, "E must be [B, N, d]");
  const int32_t B = dim(*E, 0), N = dim(*E, 1), d = dim(*E, 2), code = dtype_code(like);
  const Links l = links_of(*LC, B);
  check_lens(lens, B);
  Out LP(LPin, {B, l.m, d}, *E);
  Tensor OS;
  if (want_os) OS = Out(OSin, {B, N, d}, *E).t;
  Scope s(*E, a.object(), workspace, lime_workspace_bytes(is_xor ? LIME_OP_XOR_HISTORY : LIME_OP_LINK_HISTORY, B, N, 1, d, h, l.m, code, want_os ? 1 : 0));
  if (is_xor)
    call(lime_xor_history, ptr(E), ints(lens), ptr(LC), l.stride, ptr(Wq), ptr(Wk), ptr(Wv), ptr(&LP.t), want_os ? OS.data_ptr() : nullptr,
         B, N, d, h, l.m, scale, code, s.ws(), s.bytes(), s.stream());
  else
    call(lime_link_history, ptr(E), ints(lens), ptr(LC), l.stride, ptr(Wq), ptr(Wk), ptr(Wv), ptr(&LP.t), B, N, d, h, l.m, scale, code,
         s.ws(), s.bytes(), s.stream());
  return pair(LP.t, want_os ? &OS : nullptr);
}

// (E, lens, LC, Wq, Wk, Wv, Wu, Wo, h, scale, LP, workspace, stream) -> LP
PyObject* xor_layers(Args a) {
  const Tensor *E = a.tensor(), *lens = a.tensor(false), *LC = a.tensor(), *Wq = a.tensor(false), *Wk = a.tensor(false), *Wv = a.tensor(false),
               *Wu = a.tensor(), *Wo = a.tensor();
  const int32_t h = a.integer();
  const float scale = a.number();
  const Tensor *LPin = a.tensor(false), *workspace = a.tensor(false);
  const Tensor& like = check({E, LC, Wq, Wk, Wv, Wu, Wo, LPin});
  want_dims(*E, 3, "E must be [B, N, d]");
  const int32_t B = dim(*E, 0), N = dim(*E, 1), d = dim(*E, 2), code = dtype_code(like);
  const Links l = links_of(*LC, B);
  if (Wu->dim() != 3 || Wu->sizes() != Wo->sizes() || Wu->size(1) != d || Wu->size(2) != d)
    raise(PyExc_ValueError, "Wu and Wo must both be [n_layers, d, d]");
  check_lens(lens, B);
  Out LP(LPin, {B, l.m, d}, *E);
  Scope s(*E, a.object(), workspace, lime_workspace_bytes(LIME_OP_XOR_LAYERS, B, N, 1, d, h, l.m, code, 0));
  call(lime_xor_layers, ptr(E), ints(lens), ptr(LC), l.stride, ptr(Wq), ptr(Wk), ptr(Wv), ptr(Wu), ptr(Wo), dim(*Wu, 0), ptr(&LP.t), B, N,
       d, h, l.m, scale, code, s.ws(), s.bytes(), s.stream());
  return wrap(LP.t);
}

// (T, L, LP, Wq, Wk, Wv, h, scale, O, workspace, stream) -> O
PyObject* score_candidates(Args a) {
  const Tensor *T = a.tensor(), *L = a.tensor(), *LP = a.tensor(), *Wq = a.tensor(false), *Wk = a.tensor(false), *Wv = a.tensor(false);
  const int32_t h = a.integer();
  const float scale = a.number();
  const Tensor *Oin = a.tensor(false), *workspace = a.tensor(false);
  const Tensor& like = check({T, L, LP, Wq, Wk, Wv, Oin});
  want_dims(*T, 3, "T must be [B, C, d]");
  const int32_t B = dim(*T, 0), C = dim(*T, 1), d = dim(*T, 2), m = dim(*L, 0), code = dtype_code(like);
  Out O(Oin, T->sizes(), *T);
  Scope s(*T, a.object(), workspace, lime_workspace_bytes(LIME_OP_SCORE_CANDIDATES, B, 1, C, d, h, m, code, 0));
  call(lime_score_candidates, ptr(T), ptr(L), ptr(LP), ptr(Wq), ptr(Wk), ptr(Wv), ptr(&O.t), B, C, d, h, m, scale, code, s.ws(), s.bytes(),
       s.stream());
  return wrap(O.t);
}

// (T, E, lens, Wq, Wk, Wv, h, scale, O, workspace, stream) -> O
PyObject* target_attention(Args a) {
  const Tensor *T = a.tensor(), *E = a.tensor(), *lens = a.tensor(false), *Wq = a.tensor(false), *Wk = a.tensor(false), *Wv = a.tensor(false);
  const int32_t h = a.integer();
  const float scale = a.number();
  const Tensor *Oin = a.tensor(false), *workspace = a.tensor(false);
  const Tensor& like = check({T, E, Wq, Wk, Wv, Oin});
  want_dims(*T, 3, "T must be [B, C, d]"), want_dims(*E, 3, "E must be [B, N, d]");
  const int32_t B = dim(*T, 0), C = dim(*T, 1), d = dim(*T, 2), N = dim(*E, 1), code = dtype_code(like);
  check_lens(lens, B);
  Out O(Oin, T->sizes(), *T);
  Scope s(*T, a.object(), workspace, lime_workspace_bytes(LIME_OP_MHA_TARGET, B, N, C, d, h, 1, code, 0));
  call(mha_target_attention, ptr(T), ptr(E), ints(lens), ptr(Wq), ptr(Wk), ptr(Wv), ptr(&O.t), B, C, N, d, h, scale, code, s.ws(),
       s.bytes(), s.stream());
  return wrap(O.t);
}

// (W, ids or None, LP, Wv, O, workspace, stream) -> O; W is [B, C, h, m], with ids the table [n_items, h, m]
PyObject* score_cached(Args a) {
  const Tensor *W = a.tensor(), *ids = a.tensor(false), *LP = a.tensor(), *Wv = a.tensor(false), *Oin = a.tensor(false), *workspace = a.tensor(false);
  const Tensor& like = check({W, LP, Wv, Oin});
  want_dims(*W, ids != nullptr ? 3 : 4, ids != nullptr ? "Wtable must be [n_items, h, m]" : "W must be [B, C, h, m]");
  want_dims(*LP, 3, "LP must be [B, m, d]");
  if (ids != nullptr) {
    if (ids->scalar_type() != at::kInt || !ids->is_contiguous() || ids->device() != W->device())
      raise(PyExc_AssertionError, "ids: contiguous int32 on the device");
    want_dims(*ids, 2, "ids must be [B, C]");
  }
  const int32_t B = ids != nullptr ? dim(*ids, 0) : dim(*W, 0), C = ids != nullptr ? dim(*ids, 1) : dim(*W, 1);
  const int32_t h = dim(*W, ids != nullptr ? 1 : 2), m = dim(*W, ids != nullptr ? 2 : 3), d = dim(*LP, 2), code = dtype_code(like);
  Out O(Oin, {B, C, d}, *W);
  Scope s(*W, a.object(), workspace, lime_workspace_bytes(LIME_OP_SCORE_CACHED, B, 1, C, d, h, m, code, 0));
  if (ids != nullptr)
    call(lime_score_candidates_gathered, ptr(W), ints(ids), dim(*W, 0), ptr(LP), ptr(Wv), ptr(&O.t), B, C, d, h, m, code, s.ws(), s.bytes(),
         s.stream());
  else
    call(lime_score_candidates_cached, ptr(W), ptr(LP), ptr(Wv), ptr(&O.t), B, C, d, h, m, code, s.ws(), s.bytes(), s.stream());
  return wrap(O.t);
}

// (E, lens, prepared, h, m, scale, xor, LP, workspace, stream) -> LP
PyObject* history_prepared(Args a) {
  const Tensor *E = a.tensor(), *lens = a.tensor(false), *prepared = a.tensor(false);
  const int32_t h = a.integer(), m = a.integer();
  const float scale = a.number();
  const bool is_xor = a.truth();
  const Tensor *LPin = a.tensor(false), *workspace = a.tensor(false);
  const Tensor& like = check({E, LPin});
  want_dims(*E, 3, "E must be [B, N, d]");
  const int32_t B = dim(*E, 0), N = dim(*E, 1), d = dim(*E, 2), code = dtype_code(like);
  Out LP(LPin, {B, m, d}, *E);
  Scope s(*E, a.object(), workspace, lime_workspace_bytes(LIME_OP_LINK_HISTORY, B, N, 1, d, h, m, code, 0));
  call(lime_link_history_prepared, ptr(E), ints(lens), ptr(prepared), ptr(&LP.t), B, N, d, h, m, scale, is_xor, code, s.ws(), s.bytes(),
       s.stream());
  return wrap(LP.t);
}

// (T, LP, Wv, prepared, h, scale, O, workspace, stream) -> O
PyObject* candidates_prepared(Args a) {
  const Tensor *T = a.tensor(), *LP = a.tensor(), *Wv = a.tensor(false), *prepared = a.tensor(false);
  const int32_t h = a.integer();
  const float scale = a.number();
  const Tensor *Oin = a.tensor(false), *workspace = a.tensor(false);
  const Tensor& like = check({T, LP, Wv, Oin});
  want_dims(*T, 3, "T must be [B, C, d]"), want_dims(*LP, 3, "LP must be [B, m, d]");
  const int32_t B = dim(*T, 0), C = dim(*T, 1), d = dim(*T, 2), m = dim(*LP, 1), code = dtype_code(like);
  Out O(Oin, T->sizes(), *T);
  Scope s(*T, a.object(), workspace, lime_workspace_bytes(LIME_OP_SCORE_CANDIDATES, B, 1, C, d, h, m, code, 0));
  call(lime_score_candidates_prepared, ptr(T), ptr(LP), ptr(Wv), ptr(prepared), ptr(&O.t), B, C, d, h, m, scale, code, s.ws(), s.bytes(),
       s.stream());
  return wrap(O.t);
}

// (E, lens, LC, Wq_hist, Wk_hist, Wv_hist, T, L, Wq_cand, Wk_cand, Wv_cand, h, scale_hist, scale_cand, xor, LP, O, on_static,
//  workspace, stream) -> (LP, O)
PyObject* request(Args a) {
  const Tensor *E = a.tensor(), *lens = a.tensor(false), *LC = a.tensor(), *Wqh = a.tensor(false), *Wkh = a.tensor(false), *Wvh = a.tensor(false);
  const Tensor *T = a.tensor(), *L = a.tensor(), *Wqc = a.tensor(false), *Wkc = a.tensor(false), *Wvc = a.tensor(false);
  const int32_t h = a.integer();
  const float sh = a.number(), sc = a.number();
  const bool is_xor = a.truth();
  const Tensor *LPin = a.tensor(false), *Oin = a.tensor(false);
  const bool on_static = a.truth();
  const Tensor* workspace = a.tensor(false);
  const Tensor& like = check({E, LC, Wqh, Wkh, Wvh, T, L, Wqc, Wkc, Wvc, LPin, Oin});
  want_dims(*E, 3, "E must be [B, N, d]"), want_dims(*T, 3, "T must be [B, C, d]");
  const int32_t B = dim(*E, 0), N = dim(*E, 1), d = dim(*E, 2), C = dim(*T, 1), code = dtype_code(like);
  const Links l = links_of(*LC, B);
  check_lens(lens, B);
  Out LP(LPin, {B, l.m, d}, *E), O(Oin, T->sizes(), *T);
  if (on_static) {
    c10::DeviceGuard guard(E->device());
    void* stream = stream_handle(a.object(), E->device().index());
    call(lime_request_static, ptr(E), ints(lens), ptr(LC), l.stride, ptr(Wqh), ptr(Wkh), ptr(Wvh), ptr(T), ptr(L), ptr(Wqc), ptr(Wkc),
         ptr(Wvc), ptr(&LP.t), ptr(&O.t), B, N, C, d, h, l.m, sh, sc, is_xor, code, stream);
  } else {
    Scope s(*E, a.object(), workspace, lime_workspace_bytes(LIME_OP_REQUEST, B, N, C, d, h, l.m, code, 0));
    call(lime_request, ptr(E), ints(lens), ptr(LC), l.stride, ptr(Wqh), ptr(Wkh), ptr(Wvh), ptr(T), ptr(L), ptr(Wqc), ptr(Wkc), ptr(Wvc),
         ptr(&LP.t), ptr(&O.t), B, N, C, d, h, l.m, sh, sc, is_xor, code, s.ws(), s.bytes(), s.stream());
  }
  return pair(LP.t, &O.t);
}

// (E, lens, T, Wv, prepared, h, m, scale_hist, scale_cand, xor, LP, O, workspace, stream) -> (LP, O)
PyObject* request_prepared(Args a) {
  const Tensor *E = a.tensor(), *lens = a.tensor(false), *T = a.tensor(), *Wv = a.tensor(false), *prepared = a.tensor(false);
  const int32_t h = a.integer(), m = a.integer();
  const float sh = a.number(), sc = a.number();
  const bool is_xor = a.truth();
  const Tensor *LPin = a.tensor(false), *Oin = a.tensor(false), *workspace = a.tensor(false);
  const Tensor& like = check({E, T, Wv, LPin, Oin});
  want_dims(*E, 3, "E must be [B, N, d]"), want_dims(*T, 3, "T must be [B, C, d]");
  const int32_t B = dim(*E, 0), N = dim(*E, 1), d = dim(*E, 2), C = dim(*T, 1), code = dtype_code(like);
  check_lens(lens, B);
  Out LP(LPin, {B, m, d}, *E), O(Oin, T->sizes(), *T);
  Scope s(*E, a.object(), workspace, lime_workspace_bytes(LIME_OP_REQUEST_PREPARED, B, N, C, d, h, m, code, 0));
  call(lime_request_prepared, ptr(E), ints(lens), ptr(T), ptr(Wv), ptr(prepared), ptr(&LP.t), ptr(&O.t), B, N, C, d, h, m, sh, sc, is_xor,
       code, s.ws(), s.bytes(), s.stream());
  return pair(LP.t, &O.t);
}

// (QS, KS, VS, QT, KT, VT, dOT, dOS, lens, h, scale, workspace, stream) -> (dQS, dKS, dVS, dQT, dKT, dVT)
PyObject* xor_backward(Args a) {
  const Tensor *QS = a.tensor(), *KS = a.tensor(), *VS = a.tensor(), *QT = a.tensor(), *KT = a.tensor(), *VT = a.tensor(), *dOT = a.tensor(),
               *dOS = a.tensor(false), *lens = a.tensor(false);
  const int32_t h = a.integer();
  const float scale = a.number();
  const Tensor* workspace = a.tensor(false);
  const Tensor& like = check({QS, KS, VS, QT, KT, VT, dOT, dOS});
  want_dims(*QS, 3, "QS must be [B, N, d]");
  const int32_t B = dim(*QS, 0), N = dim(*QS, 1), d = dim(*QS, 2), code = dtype_code(like);
  if (QT->dim() != 3 || QT->size(0) != B) raise(PyExc_ValueError, "the projected links must be per user: [B, m, d]");
  const int32_t m = dim(*QT, 1);
  check_lens(lens, B);
  std::array<Tensor, 6> o;
  for (int i = 0; i < 6; ++i) o[i] = at::empty(i < 3 ? QS->sizes() : QT->sizes(), QS->options());
  Scope s(*QS, a.object(), workspace, lime_workspace_bytes(LIME_OP_XOR_BACKWARD, B, N, 1, d, h, m, code, 0));
  call(lime_xor_backward, ptr(QS), ptr(KS), ptr(VS), ptr(QT), ptr(KT), ptr(VT), ptr(dOT), ptr(dOS), ints(lens), ptr(&o[0]), ptr(&o[1]),
       ptr(&o[2]), ptr(&o[3]), ptr(&o[4]), ptr(&o[5]), B, N, m, d, h, scale, code, s.ws(), s.bytes(), s.stream());
  PyObject* t = PyTuple_New(6);
  if (t == nullptr) throw PyFailed{};
  for (int i = 0; i < 6; ++i) PyTuple_SET_ITEM(t, i, wrap(o[i]));
  return t;
}

// (model, E, lens, EC, T, want_intermediates, workspace, stream) -> scores, or (scores, LC, LP, O); model: a lime_scoring_model
// through the buffer protocol
PyObject* scores(Args a) {
  struct Buffer {
    Py_buffer b;
    explicit Buffer(PyObject* o) {
      if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) throw PyFailed{};
    }
    ~Buffer() { PyBuffer_Release(&b); }
  } model(a.object());
  if (model.b.len != static_cast<Py_ssize_t>(sizeof(lime_scoring_model))) raise(PyExc_TypeError, "model must be a ScoringModel");
  const lime_scoring_model* M = static_cast<const lime_scoring_model*>(model.b.buf);
  const Tensor *E = a.tensor(), *lens = a.tensor(false), *EC = a.tensor(), *T = a.tensor();
  const bool want = a.truth();
  const Tensor* workspace = a.tensor(false);
  const Tensor& like = check({E, EC, T});
  want_dims(*E, 3, "E must be [B, N, d]"), want_dims(*T, 3, "T must be [B, C, d]");
  const int32_t B = dim(*E, 0), N = dim(*E, 1), d = dim(*E, 2), C = dim(*T, 1), code = dtype_code(like);
  check_lens(lens, B);
  const Tensor out = at::empty({B, C}, E->options().dtype(at::kFloat));
  Tensor LC, LP, O;
  if (want) LC = at::empty({B, M->m, d}, E->options()), LP = at::empty({B, M->m, d}, E->options()), O = at::empty(T->sizes(), T->options());
  const size_t need = lime_scores_workspace_bytes(M, B, N, C, code);
  if (need == 0) lime_failed(LIME_INVALID_ARG, "lime_scores: the model or the sizes are not valid");
  Scope s(*E, a.object(), workspace, need);
  call(lime_scores, M, ptr(E), ints(lens), ptr(EC), ptr(T), want ? LC.data_ptr() : nullptr, want ? LP.data_ptr() : nullptr,
       want ? O.data_ptr() : nullptr, static_cast<float*>(out.data_ptr()), B, N, C, code, s.ws(), s.bytes(), s.stream());
  if (!want) return wrap(out);
  PyObject* t = PyTuple_New(4);
  if (t == nullptr) throw PyFailed{};
  PyTuple_SET_ITEM(t, 0, wrap(out)), PyTuple_SET_ITEM(t, 1, wrap(LC)), PyTuple_SET_ITEM(t, 2, wrap(LP)), PyTuple_SET_ITEM(t, 3, wrap(O));
  return t;
}

// (bytes, device index, stream or None) -> the shared workspace of that device and stream
PyObject* workspace(Args a) {
  const size_t bytes = PyLong_AsSize_t(a.object());
  if (PyErr_Occurred()) throw PyFailed{};
  const int device = a.integer();
  return wrap(shared_workspace(bytes, at::Device(at::kCUDA, static_cast<c10::DeviceIndex>(device)), stream_handle(a.object(), device)));
}

// (LimeError)
PyObject* set_error_type(Args a) {
  PyObject* type = a.object();
  Py_INCREF(type);
  Py_XDECREF(g_lime_error);
  g_lime_error = type;
  Py_RETURN_NONE;
}

template <PyObject* (*F)(Args), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS  // (torch's own: out of memory and the like)
  try {
    return F(Args(args, n, N));
  } catch (const PyFailed&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

#define LIME_ENTRY(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {LIME_ENTRY(history, 14), LIME_ENTRY(xor_layers, 13), LIME_ENTRY(score_candidates, 11), LIME_ENTRY(target_attention, 11),
                           LIME_ENTRY(score_cached, 7), LIME_ENTRY(history_prepared, 10), LIME_ENTRY(candidates_prepared, 9),
                           LIME_ENTRY(request, 20), LIME_ENTRY(request_prepared, 14), LIME_ENTRY(xor_backward, 13), LIME_ENTRY(scores, 8),
                           LIME_ENTRY(workspace, 3), LIME_ENTRY(set_error_type, 1), {nullptr, nullptr, 0, nullptr}};
#undef LIME_ENTRY
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_lime_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lime_torch() { return PyModule_Create(&g_module); }
