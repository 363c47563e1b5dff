// What binding.py's entry points do per call, in native code: reads the arguments, allocates the outputs and the workspace with
// torch's allocator and calls the C ABI of umas.h.  The entry points themselves (names, defaults, errors, results) are
// binding.py's; a call here returns its outputs, or the status (an int) when the library refuses.
// In Python most of a small call went into this: 27 tensors at 1.3 us, a pointer at 0.5 to 1 us each, structs of pointers and the
// current stream (2.9 us): routing, advantages, KL, whitening and the ready batch of 40 000 tokens took 139 us to issue, 54 of them
// in the library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/TensorOptions.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <initializer_list>

#include "../../include/umas.h"

namespace {

struct Failed {};   // a Python error is set

// ------------------------------------------------------------------ arguments
[[noreturn]] void type_error(const char* what, PyObject* got) {
  PyErr_Format(PyExc_TypeError, "%s expected, got %s", what, Py_TYPE(got)->tp_name);
  throw Failed();
}
// anything with __index__ (Python's and numpy's integers), no floats; more bits than fit are cut off
int64_t integer(PyObject* o) {
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
  if (v == static_cast<unsigned long long>(-1) && PyErr_Occurred()) throw Failed();
  return static_cast<int64_t>(v);
}
int32_t integer32(PyObject* o) { return static_cast<int32_t>(integer(o)); }
int64_t as_int(PyObject* o) {                             // int(o)
  PyObject* n = PyNumber_Long(o);
  if (!n) throw Failed();
  const int64_t v = integer(n);
  Py_DECREF(n);
  return v;
}
float real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Failed();
  return static_cast<float>(v);
}
int truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Failed();
  return v;
}
void* stream_of(PyObject* o) { return reinterpret_cast<void*>(static_cast<uintptr_t>(integer(o))); }

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) type_error("tensor", o);
  return THPVariable_Unpack(o);
}
template <class T>
T* ptr(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }
template <class T>
T* ptr_or_null(PyObject* o) { return o == Py_None ? nullptr : ptr<T>(tensor(o)); }
// pointers of arrays that may be empty: an empty tensor has no storage, the ABI wants non-NULL pointers even for size 0
template <class T>
T* ptr_or(const at::Tensor& t, void* otherwise) {
  T* p = ptr<T>(t);
  return p ? p : static_cast<T*>(otherwise);
}
int dtype_code(PyObject* o) {
  const at::Tensor& t = tensor(o);
  if (t.scalar_type() == at::kFloat) return UMAS_F32;
  if (t.scalar_type() == at::kBFloat16) return UMAS_BF16;
  PyObject* dt = PyObject_GetAttrString(o, "dtype");
  if (dt) PyErr_Format(PyExc_TypeError, "unsupported dtype %S", dt);
  Py_XDECREF(dt);
  throw Failed();
}
struct Rows {                                             // [n, d] hidden states
  const at::Tensor& t;
  int dt;
  int64_t n;
  int32_t d;
  explicit Rows(PyObject* o) : t(tensor(o)) {
    if (t.dim() != 2) {
      PyErr_Format(PyExc_ValueError, "H must have two dimensions, not %d", static_cast<int>(t.dim()));
      throw Failed();
    }
    n = t.size(0);
    d = static_cast<int32_t>(t.size(1));
    dt = dtype_code(o);
  }
};
struct Selection {                                        // None: all rows; an empty one still needs a pointer
  const int32_t* p = nullptr;
  int64_t n;
  Selection(PyObject* o, int64_t all, void* otherwise = nullptr) : n(all) {
    if (o == Py_None) return;
    const at::Tensor& t = tensor(o);
    n = t.numel();
    p = ptr_or<const int32_t>(t, otherwise);
  }
  void point(void* otherwise, PyObject* o) { if (o != Py_None && !p) p = static_cast<const int32_t*>(otherwise); }
};

PyObject* ascontiguousarray = nullptr;                    // numpy's
// A host array of the ABI's type: the object's own memory where it has that type, is contiguous and lies at a multiple of the type's
// size, else numpy's copy.
struct HostArray {
  Py_buffer view{};
  bool held = false;
  int64_t len = 0;                                        // of the first dimension
  HostArray() = default;
  HostArray(const HostArray&) = delete;
  ~HostArray() { if (held) PyBuffer_Release(&view); }
  void get(PyObject* o, char kind, int size, const char* np_type) {
    if (o == Py_None) return;
    if (PyBytes_Check(o) || !(PyObject_CheckBuffer(o) && take(o, kind, size))) {   // bytes: text to numpy
      PyErr_Clear();
      PyObject* a = PyObject_CallFunction(ascontiguousarray, "Os", o, np_type);
      if (!a) throw Failed();
      bool ok = take(a, kind, size);                      // the view holds the array
      if (!ok) {                                          // the right type and contiguous, but not aligned
        PyErr_Clear();
        PyObject* const c = PyObject_CallMethod(a, "copy", nullptr);
        Py_DECREF(a);
        if (!(a = c)) throw Failed();
        ok = take(a, kind, size);
      }
      Py_DECREF(a);
      if (!ok) {
        if (!PyErr_Occurred()) PyErr_Format(PyExc_TypeError, "array of %s expected", np_type);
        throw Failed();
      }
    }
    len = view.ndim > 0 ? view.shape[0] : 1;                // a single number: one entry
  }
  template <class T>
  const T* as() const { return held ? static_cast<const T*>(view.buf) : nullptr; }

 private:
  bool take(PyObject* o, char kind, int size) {           // kind: i(nteger), u(nsigned), f(loat)
    if (PyObject_GetBuffer(o, &view, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) return false;
    const char* f = view.format;
    bool ok = f && f[0] && !f[1] && view.itemsize == size && reinterpret_cast<uintptr_t>(view.buf) % size == 0;
    if (ok) ok = kind == 'i' ? f[0] == 'i' || f[0] == 'l' || f[0] == 'q' : kind == 'u' ? f[0] == 'B' : f[0] == 'f';
    if (!ok) PyBuffer_Release(&view);
    held = ok;
    return ok;
  }
};
#define I32_ARRAY(name, obj) HostArray name; name.get(obj, 'i', 4, "int32")
#define I64_ARRAY(name, obj) HostArray name; name.get(obj, 'i', 8, "int64")
#define F32_ARRAY(name, obj) HostArray name; name.get(obj, 'f', 4, "float32")
#define U8_ARRAY(name, obj) HostArray name; name.get(obj, 'u', 1, "uint8")

// ------------------------------------------------------------------ outputs
at::Tensor fresh(at::IntArrayRef size, at::ScalarType type, const at::Device& dev) {
  return at::empty(size, at::TensorOptions().dtype(type).device(dev));
}
at::Tensor workspace(size_t bytes, const at::Device& dev) {
  return fresh({static_cast<int64_t>(std::max<size_t>(bytes, 256))}, at::kByte, dev);
}
struct Output {                                           // what the caller passed, or a new tensor
  at::Tensor t;
  PyObject* given;
  template <class Make>
  Output(PyObject* o, Make make) : given(o == Py_None ? nullptr : o) { t = given ? tensor(o) : make(); }
  PyObject* object() const {
    if (!given) return THPVariable_Wrap(t);
    Py_INCREF(given);
    return given;
  }
};
PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }
PyObject* pack(std::initializer_list<PyObject*> items) {  // takes the references
  bool ok = true;
  for (PyObject* o : items) ok = ok && o;
  PyObject* r = ok ? PyTuple_New(static_cast<Py_ssize_t>(items.size())) : nullptr;
  if (!r) {
    for (PyObject* o : items) Py_XDECREF(o);
    return nullptr;
  }
  Py_ssize_t i = 0;
  for (PyObject* o : items) PyTuple_SET_ITEM(r, i++, o);
  return r;
}
struct Unlocked {                                         // the interpreter lock is taken again also when the call throws
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class Call>
umas_status unlocked(Call call) {                         // the library needs no Python
  const Unlocked without_lock;
  return call();
}
#define UMAS_CALL(...)                                                        \
  do {                                                                        \
    const umas_status s__ = unlocked([&] { return __VA_ARGS__; });            \
    if (s__ != UMAS_OK) return PyLong_FromLong(static_cast<long>(s__));       \
  } while (0)

constexpr int kStreamTensors = 16;
const char* const kStreamNames[kStreamTensors] = {"model_tok_off", "perm", "tok_turn", "tok_role", "tok_mask", "tok_reward", "turn_seg_off",
                                                  "seg_turn", "model_turn_off", "traj_seg_off", "model_trajrun_off", "rowsel",
                                                  "model_rowsel_off", "turn_scalar", "turn_step", "tok_flags"};
static_assert(sizeof(umas_streams) == kStreamTensors * sizeof(void*), "one pointer per name");
PyObject* g_stream_names[kStreamTensors];
PyObject *g_n_tokens, *g_n_turns, *g_n_models;

struct Ref {                                              // an owned reference
  PyObject* o;
  explicit Ref(PyObject* p) : o(p) { if (!p) throw Failed(); }
  Ref(const Ref&) = delete;
  ~Ref() { Py_DECREF(o); }
};
// the ABI's struct of a Streams object; the object keeps its tensors
umas_streams streams_of(PyObject* o, void* otherwise) {
  umas_streams s;
  void** p = reinterpret_cast<void**>(&s);
  for (int i = 0; i < kStreamTensors; ++i) {
    const Ref t(PyObject_GetAttr(o, g_stream_names[i]));
    p[i] = ptr_or<void>(tensor(t.o), otherwise);
  }
  return s;
}
int64_t int_attr(PyObject* o, PyObject* name) { const Ref v(PyObject_GetAttr(o, name)); return integer(v.o); }
at::Device device_of(PyObject* streams, int field) { const Ref t(PyObject_GetAttr(streams, g_stream_names[field])); return tensor(t.o).device(); }
constexpr int kTokReward = 5, kRowsel = 11;

// ------------------------------------------------------------------ entry points
PyObject* assign(PyObject* const* a) {
  umas_graph g;
  umas_rewards r;
  g.n_roles = integer32(a[0]);
  g.n_models = integer32(a[1]);
  for (int i : {3, 5})                                    // offsets have a length
    if (a[i] != Py_None && PyObject_Size(a[i]) < 0) throw Failed();
  I32_ARRAY(role_to_model, a[2]);
  I32_ARRAY(traj_turn_off, a[3]);
  I32_ARRAY(turn_role, a[4]);
  I64_ARRAY(turn_tok_off, a[5]);
  const at::Tensor& mask = tensor(a[6]);
  I32_ARRAY(turn_pred_off, a[7]);
  I32_ARRAY(turn_pred, a[8]);
  I32_ARRAY(traj_group, a[9]);
  F32_ARRAY(role_reward, a[10]);
  F32_ARRAY(turn_reward, a[11]);
  F32_ARRAY(traj_reward, a[12]);
  F32_ARRAY(w_role, a[13]);
  F32_ARRAY(w_turn, a[14]);
  F32_ARRAY(w_traj, a[15]);
  r.place_mode = integer32(a[16]);
  r.norm_eps = real(a[17]);
  void* const st = stream_of(a[18]);
  const int64_t N = mask.numel(), U = turn_tok_off.len - 1, M = g.n_models;
  g.n_traj = static_cast<int32_t>(traj_turn_off.len - 1);
  g.n_turns = static_cast<int32_t>(U);
  g.n_tokens = N;
  g.role_to_model = role_to_model.as<int32_t>();
  g.traj_turn_off = traj_turn_off.as<int32_t>();
  g.turn_role = turn_role.as<int32_t>();
  g.turn_tok_off = turn_tok_off.as<int64_t>();
  g.turn_pred_off = turn_pred_off.as<int32_t>();
  g.turn_pred = turn_pred.as<int32_t>();
  g.traj_group = traj_group.as<int32_t>();
  r.role_reward = role_reward.as<float>();
  r.turn_reward = turn_reward.as<float>();
  r.traj_reward = traj_reward.as<float>();
  r.w_role = w_role.as<float>();
  r.w_turn = w_turn.as<float>();
  r.w_traj = w_traj.as<float>();
  const at::Device dev = mask.device();
  const int64_t U1 = std::max<int64_t>(U, 1), N1 = std::max<int64_t>(N, 1);
  const auto i64 = at::kLong, i32 = at::kInt, f32 = at::kFloat, u8 = at::kByte;
  const at::Tensor out[kStreamTensors] = {
      fresh({M + 1}, i64, dev), fresh({N}, i64, dev), fresh({N}, i32, dev), fresh({N}, i32, dev), fresh({N}, u8, dev), fresh({N}, f32, dev),
      fresh({U + 1}, i64, dev), fresh({U1}, i32, dev), fresh({M + 1}, i32, dev), fresh({U + 1}, i64, dev), fresh({M + 1}, i32, dev),
      fresh({N1}, i32, dev), fresh({M + 1}, i64, dev), fresh({U1}, f32, dev), fresh({U1}, i32, dev), fresh({N}, u8, dev)};
  const at::Tensor ws = workspace(umas_assign_workspace_bytes(&g), dev);
  umas_streams s;
  for (int i = 0; i < kStreamTensors; ++i) reinterpret_cast<void**>(&s)[i] = ptr_or<void>(out[i], ws.data_ptr());
  UMAS_CALL(umas_assign_token_rewards(&g, &r, ptr_or<uint8_t>(mask, ws.data_ptr()), &s, ws.data_ptr(), ws.numel(), st));
  PyObject* res = PyTuple_New(3 + kStreamTensors);
  if (!res) return nullptr;
  PyTuple_SET_ITEM(res, 0, PyLong_FromLongLong(N));
  PyTuple_SET_ITEM(res, 1, PyLong_FromLongLong(U));
  PyTuple_SET_ITEM(res, 2, PyLong_FromLongLong(M));
  for (int i = 0; i < kStreamTensors; ++i) PyTuple_SET_ITEM(res, 3 + i, wrap(out[i]));
  return res;
}

PyObject* advantages(PyObject* const* a) {                // streams, value, gamma, lam, gamma_turn, seg_mode, stream
  const at::Device dev = device_of(a[0], kTokReward);
  const int64_t N = int_attr(a[0], g_n_tokens);
  const int32_t U = static_cast<int32_t>(int_attr(a[0], g_n_turns));
  const float gamma = real(a[2]), lam = real(a[3]), gamma_turn = real(a[4]);
  const int32_t seg = integer32(a[5]);
  const at::Tensor adv = fresh({N}, at::kFloat, dev), ret = fresh({N}, at::kFloat, dev), ws = workspace(umas_advantages_workspace_bytes(N), dev);
  const umas_streams s = streams_of(a[0], ws.data_ptr());
  const float* value = ptr_or_null<const float>(a[1]);
  void* const st = stream_of(a[6]);
  UMAS_CALL(umas_advantages(&s, N, U, value, gamma, lam, gamma_turn, seg, ptr<float>(adv), ptr<float>(ret), ws.data_ptr(), ws.numel(), st));
  return pack({wrap(adv), wrap(ret)});
}

PyObject* policy_logprobs(PyObject* const* a) {           // H, W, ids, rowsel, want_entropy, workspace, stream
  const Rows H(a[0]);
  const at::Tensor &W = tensor(a[1]), &ids = tensor(a[2]);
  const int32_t V = static_cast<int32_t>(W.size(0));
  Selection sel(a[3], H.n);
  const at::Device dev = H.t.device();
  const at::Tensor logp = fresh({H.n}, at::kFloat, dev), lse = fresh({H.n}, at::kFloat, dev);
  const bool want = truth(a[4]);
  const at::Tensor entropy = want ? fresh({H.n}, at::kFloat, dev) : at::Tensor();
  const umas_dtype dt = static_cast<umas_dtype>(H.dt);
  const Output ws(a[5], [&] { return workspace(umas_policy_logprobs_workspace_bytes(sel.n, H.d, V, dt), dev); });
  sel.point(ws.t.data_ptr(), a[3]);
  void* const st = stream_of(a[6]);
  float* const e = want ? ptr<float>(entropy) : nullptr;
  UMAS_CALL(umas_policy_logprobs(H.t.data_ptr(), W.data_ptr(), dt, H.n, H.d, V, ptr<int32_t>(ids), sel.p, sel.n, ptr<float>(logp), ptr<float>(lse), e,
                                 ws.t.data_ptr(), ws.t.numel(), st));
  if (!want) Py_INCREF(Py_None);
  return pack({wrap(logp), wrap(lse), want ? wrap(entropy) : Py_None});
}

PyObject* policy_logprobs_static(PyObject* const* a) {    // H, W, ids, rowsel, logp, lse, entropy, stream
  const Rows H(a[0]);
  const at::Tensor &W = tensor(a[1]), &ids = tensor(a[2]);
  const at::Device dev = H.t.device();
  auto row = [&] { return fresh({H.n}, at::kFloat, dev); };
  const Output logp(a[4], row), lse(a[5], row), entropy(a[6], row);
  Selection sel(a[3], H.n);
  sel.point(W.data_ptr(), a[3]);
  void* const st = stream_of(a[7]);
  UMAS_CALL(umas_policy_logprobs_static(H.t.data_ptr(), W.data_ptr(), static_cast<umas_dtype>(H.dt), H.n, H.d, static_cast<int32_t>(W.size(0)),
                                        ptr<int32_t>(ids), sel.p, sel.n, ptr<float>(logp.t), ptr<float>(lse.t), ptr<float>(entropy.t), st));
  return pack({logp.object(), lse.object(), entropy.object()});
}

PyObject* ppo_loss(PyObject* const* a) {
  // H, W, ids, rowsel, logp_old, adv, tok_role, n_roles, clip_eps, entropy_coef, dual_clip, accumulate_dW, norm_rows, logp_ref, kl_coef,
  // dW, dH, logp_new, stats, workspace, stream
  const Rows H(a[0]);
  const at::Tensor &W = tensor(a[1]), &ids = tensor(a[2]), &adv = tensor(a[5]);
  const int32_t V = static_cast<int32_t>(W.size(0)), n_roles = integer32(a[7]);
  Selection sel(a[3], H.n);
  const at::Device dev = H.t.device();
  const umas_dtype dt = static_cast<umas_dtype>(H.dt);
  const Output dW(a[15], [&] { return fresh({W.size(0), H.d}, at::kFloat, dev); });
  const Output dH(a[16], [&] { return at::empty_like(H.t); });
  const Output logp_new(a[17], [&] { return fresh({H.n}, at::kFloat, dev); });
  const Output stats(a[18], [&] { return fresh({(1 + static_cast<int64_t>(n_roles)) * static_cast<int64_t>(sizeof(umas_loss_stats))}, at::kByte, dev); });
  const float clip_eps = real(a[8]), entropy_coef = real(a[9]), dual_clip = real(a[10]), kl_coef = real(a[14]);
  const Output ws(a[19], [&] {
    const auto bytes = entropy_coef > 0.f ? umas_ppo_loss_workspace_bytes_entropy : umas_ppo_loss_workspace_bytes;
    return workspace(bytes(sel.n, H.d, V, dt, n_roles), dev);
  });
  sel.point(ws.t.data_ptr(), a[3]);
  const float* const logp_old = ptr_or_null<const float>(a[4]);
  const int32_t* const role = ptr_or_null<const int32_t>(a[6]);
  const int32_t accumulate = truth(a[11]);
  const int64_t norm_rows = as_int(a[12]);
  const float* const logp_ref = ptr_or_null<const float>(a[13]);
  void* const st = stream_of(a[20]);
  UMAS_CALL(umas_ppo_loss_fwd_bwd(H.t.data_ptr(), W.data_ptr(), dt, H.n, H.d, V, ptr<int32_t>(ids), sel.p, sel.n, logp_old, ptr<float>(adv), role,
                                  n_roles, clip_eps, entropy_coef, dual_clip, accumulate, norm_rows, logp_ref, kl_coef,
                                  ptr<umas_loss_stats>(stats.t), ptr<float>(logp_new.t), dH.t.data_ptr(), ptr<float>(dW.t), ws.t.data_ptr(),
                                  ws.t.numel(), st));
  return pack({stats.object(), logp_new.object(), dH.object(), dW.object()});
}

PyObject* values(PyObject* const* a) {                    // H, w, bias, rowsel, value, stream
  const Rows H(a[0]);
  const at::Tensor& w = tensor(a[1]);
  const Output value(a[4], [&] { return fresh({H.n}, at::kFloat, H.t.device()); });
  Selection sel(a[3], H.n);
  sel.point(w.data_ptr(), a[3]);
  const float bias = real(a[2]);
  void* const st = stream_of(a[5]);
  UMAS_CALL(umas_values(H.t.data_ptr(), w.data_ptr(), bias, static_cast<umas_dtype>(H.dt), H.n, H.d, sel.p, sel.n, ptr<float>(value.t), st));
  return value.object();
}

PyObject* value_loss(PyObject* const* a) {
  // H, w, bias, rowsel, value_old, ret, tok_role, n_roles, clip_eps_v, accumulate_dH, accumulate_dw, norm_rows, dH, dw, db, value_new,
  // stats, workspace, stream
  const Rows H(a[0]);
  const at::Tensor& w = tensor(a[1]);
  const at::Device dev = H.t.device();
  const umas_dtype dt = static_cast<umas_dtype>(H.dt);
  const int32_t n_roles = integer32(a[7]);
  Selection sel(a[3], H.n);
  const Output dH(a[12], [&] { return at::empty_like(H.t); });
  const Output dw(a[13], [&] { return fresh({H.d}, at::kFloat, dev); });
  const Output db(a[14], [&] { return fresh({1}, at::kFloat, dev); });
  const Output value_new(a[15], [&] { return fresh({H.n}, at::kFloat, dev); });
  const Output stats(a[16], [&] { return fresh({(1 + static_cast<int64_t>(n_roles)) * static_cast<int64_t>(sizeof(umas_value_stats))}, at::kByte, dev); });
  const Output ws(a[17], [&] { return workspace(umas_value_workspace_bytes(sel.n, H.d, dt, n_roles), dev); });
  sel.point(ws.t.data_ptr(), a[3]);
  const float bias = real(a[2]), clip_eps = real(a[8]);
  const float *const value_old = ptr_or_null<const float>(a[4]), *const ret = ptr_or_null<const float>(a[5]);
  const int32_t* const role = ptr_or_null<const int32_t>(a[6]);
  const int32_t acc_dH = truth(a[9]), acc_dw = truth(a[10]);
  const int64_t norm_rows = as_int(a[11]);
  void* const st = stream_of(a[18]);
  UMAS_CALL(umas_value_loss_fwd_bwd(H.t.data_ptr(), w.data_ptr(), bias, dt, H.n, H.d, sel.p, sel.n, value_old, ret, role, n_roles, clip_eps, acc_dH,
                                    acc_dw, norm_rows, ptr<umas_value_stats>(stats.t), ptr<float>(value_new.t), dH.t.data_ptr(),
                                    ptr<float>(dw.t), ptr<float>(db.t), ws.t.data_ptr(), ws.t.numel(), st));
  return pack({stats.object(), value_new.object(), dH.object(), dw.object(), db.object()});
}

PyObject* kl_rewards(PyObject* const* a) {                // tok_reward, logp, logp_ref, tok_mask, beta, out, stream
  const at::Tensor& r = tensor(a[0]);
  const int64_t n = r.numel();
  const at::Device dev = r.device();
  const Output out(a[5], [&] { return at::empty_like(r); });
  const at::Tensor kl = fresh({1}, at::kFloat, dev), ws = workspace(umas_kl_rewards_workspace_bytes(n), dev);
  auto at_ = [&](const at::Tensor& t) { return n ? t.data_ptr() : ws.data_ptr(); };
  const at::Tensor &logp = tensor(a[1]), &ref = tensor(a[2]), &mask = tensor(a[3]);
  const float beta = real(a[4]);
  void* const st = stream_of(a[6]);
  UMAS_CALL(umas_kl_rewards(static_cast<float*>(at_(r)), static_cast<float*>(at_(logp)), static_cast<float*>(at_(ref)), static_cast<uint8_t*>(at_(mask)), n,
                            beta, static_cast<float*>(at_(out.t)), ptr<float>(kl), ws.data_ptr(), ws.numel(), st));
  return pack({out.object(), wrap(kl)});
}

PyObject* whiten(PyObject* const* a) {                    // adv, tok_mask, tok_role, model_tok_off, n_roles, scope, eps, out, stream
  const at::Tensor& adv = tensor(a[0]);
  const int64_t n = adv.numel();
  const at::Device dev = adv.device();
  I64_ARRAY(off, a[3]);
  const int32_t n_models = static_cast<int32_t>(off.len - 1), n_roles = integer32(a[4]), scope = integer32(a[5]);
  const Output out(a[7], [&] { return at::empty_like(adv); });
  const at::Tensor ws = workspace(umas_whiten_workspace_bytes(n, n_models, n_roles), dev);
  auto at_ = [&](PyObject* o) -> void* { return o == Py_None ? nullptr : n ? tensor(o).data_ptr() : ws.data_ptr(); };
  const float eps = real(a[6]);
  const float* const x = static_cast<float*>(at_(a[0]));
  const uint8_t* const mask = static_cast<uint8_t*>(at_(a[1]));
  const int32_t* const role = static_cast<int32_t*>(at_(a[2]));
  float* const y = static_cast<float*>(n ? out.t.data_ptr() : ws.data_ptr());
  void* const st = stream_of(a[8]);
  UMAS_CALL(umas_whiten_advantages(x, mask, role, off.as<int64_t>(), n_models, n_roles, n, scope, eps, y, ws.data_ptr(), ws.numel(), st));
  return out.object();
}

PyObject* ready_batch(PyObject* const* a) {               // streams, traj_turn_off, cut, parts or rows, keep, order, stream
  const at::Device dev = device_of(a[0], kRowsel);
  I32_ARRAY(tto, a[1]);
  const int32_t cut = integer32(a[2]);                    // 0: by trajectories, 1: by rows, 2: packed
  U8_ARRAY(keep, a[4]);
  I32_ARRAY(order, a[5]);
  const int32_t B = static_cast<int32_t>(tto.len - 1), U = static_cast<int32_t>(int_attr(a[0], g_n_turns)), M = static_cast<int32_t>(int_attr(a[0], g_n_models));
  int64_t n_rowsel;
  {
    const Ref t(PyObject_GetAttr(a[0], g_stream_names[kRowsel]));
    n_rowsel = tensor(t.o).numel();
  }
  const int64_t arg = cut == 2 ? as_int(a[3]) : integer32(a[3]);
  const at::Tensor rows = fresh({std::max<int64_t>(n_rowsel, 1)}, at::kInt, dev);
  const at::Tensor off = fresh({M, (cut == 2 ? B : arg) + 1}, at::kLong, dev);
  const at::Tensor parts = cut == 2 ? fresh({M}, at::kInt, dev) : at::Tensor();
  const at::Tensor ws = workspace(umas_ready_batch_workspace_bytes(B, M), dev);
  const umas_streams s = streams_of(a[0], ws.data_ptr());
  const int32_t* const t = tto.as<int32_t>();
  const uint8_t* const k = keep.as<uint8_t>();
  const int32_t* const o = order.as<int32_t>();
  void* const st = stream_of(a[6]);
  if (cut == 2) {
    UMAS_CALL(umas_ready_batch_packed(&s, M, U, t, B, k, o, arg, ptr<int32_t>(rows), ptr<int64_t>(off), ptr<int32_t>(parts), ws.data_ptr(), ws.numel(), st));
    return pack({wrap(rows), wrap(off), wrap(parts)});
  }
  const auto fn = cut == 1 ? umas_ready_batch_balanced : umas_ready_batch;
  UMAS_CALL(fn(&s, M, U, t, B, k, o, static_cast<int32_t>(arg), ptr<int32_t>(rows), ptr<int64_t>(off), ws.data_ptr(), ws.numel(), st));
  return pack({wrap(rows), wrap(off)});
}

// ------------------------------------------------------------------ module
template <PyObject* (*F)(PyObject* const*), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != N) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", N, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const Failed&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}
#define ENTRY(name, f, n) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&entry<f, n>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {ENTRY("assign", assign, 19), ENTRY("advantages", advantages, 7), ENTRY("policy_logprobs", policy_logprobs, 7),
                           ENTRY("policy_logprobs_static", policy_logprobs_static, 8), ENTRY("ppo_loss", ppo_loss, 21), ENTRY("values", values, 6),
                           ENTRY("value_loss", value_loss, 19), ENTRY("kl_rewards", kl_rewards, 7), ENTRY("whiten", whiten, 9),
                           ENTRY("ready_batch", ready_batch, 7), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_umas_torch", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__umas_torch() {
  PyObject* np = PyImport_ImportModule("numpy");
  if (!np) return nullptr;
  ascontiguousarray = PyObject_GetAttrString(np, "ascontiguousarray");
  Py_DECREF(np);
  if (!ascontiguousarray) return nullptr;
  for (int i = 0; i < kStreamTensors; ++i) g_stream_names[i] = PyUnicode_InternFromString(kStreamNames[i]);
  g_n_tokens = PyUnicode_InternFromString("n_tokens");
  g_n_turns = PyUnicode_InternFromString("n_turns");
  g_n_models = PyUnicode_InternFromString("n_models");
  return PyModule_Create(&g_module);
}
