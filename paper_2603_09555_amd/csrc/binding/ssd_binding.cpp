// The marshalling of paper_2603_09555_amd/ssd.py in native code: checks, outputs, pointers and the call of the C ABI for the
// ordinary case, dense device tensors of the expected types and shapes (outputs that the caller brings: of the expected
// type and large enough).  Anything else -- other tensor types, missing arguments, shapes that don't fit -- is answered with
// None before anything is allocated or enqueued, and ssd.py then goes through the call itself and raises what there is to
// raise.
//
// Why: a generation step of one layer is bound by the host.  A convolution and a decode step, kernels of 7 us together, took
// 21.9 us from Python (checks and ctypes some 5 us a call, an output tensor 1.2 to 1.8 us each, the launch 2.5).
//
// The functions of the C ABI are called through addresses that ssd.py hands over: this module links against torch alone.
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>

#include <cstdint>

#include "ssd.h"

namespace {

struct Api {
  decltype(&ssd_prefill_workspace_bytes) prefill_workspace_bytes;
  decltype(&ssd_prefill) prefill;
  decltype(&ssd_prefill_dt) prefill_dt;
  decltype(&ssd_prefill_varlen_workspace_bytes) varlen_workspace_bytes;
  decltype(&ssd_prefill_varlen) varlen;
  decltype(&ssd_prefill_varlen_dt) varlen_dt;
  decltype(&ssd_decode_step) decode_step;
  decltype(&ssd_decode_step_layers) decode_layers;
  decltype(&ssd_decode_step_layers_dt) decode_layers_dt;
  decltype(&ssd_decode_steps_layers) decode_steps;
  decltype(&ssd_decode_steps_layers_dt) decode_steps_dt;
  decltype(&ssd_conv1d_prefill) conv_prefill;
  decltype(&ssd_conv1d_step) conv_step;
} api;

// An argument: a plain dense device tensor, or None.
struct Arg {
  const at::Tensor *t = nullptr;
  bool ok = false;
  void *ptr() const { return t != nullptr ? t->data_ptr() : nullptr; }
};
Arg tensor(PyObject *o) {
  Arg a;
  if (THPVariable_CheckExact(o)) {
    a.t = &THPVariable_Unpack(o);
    a.ok = a.t->is_cuda() && a.t->layout() == at::kStrided && a.t->is_contiguous();
  }
  return a;
}
Arg tensor_or_none(PyObject *o) {
  if (o != Py_None) return tensor(o);
  Arg a;
  a.ok = true;
  return a;
}
bool is(const Arg &a, std::initializer_list<int64_t> shape) { return a.t->sizes() == at::IntArrayRef(shape); }
bool f32(const Arg &a) { return a.t->scalar_type() == at::kFloat; }
// an fp32 vector of (at least) that many values, whatever its shape
bool f32_of(const Arg &a, int64_t values) { return f32(a) && a.t->numel() >= values; }
// SSD_F32, SSD_BF16 or -1
int io_of(const Arg &a) {
  const auto d = a.t->scalar_type();
  return d == at::kBFloat16 ? SSD_BF16 : d == at::kFloat ? SSD_F32 : -1;
}
bool fits(std::initializer_list<int64_t> values) {
  for (int64_t v : values)
    if (v < 0 || v > INT32_MAX) return false;
  return true;
}
void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// dt_bias, dt_softplus, dt_limit as three arguments; `given`: any of them asks for the transform.
struct DtArgs {
  ssd_dt_transform x = {};
  bool ok = false, given = false;
};
DtArgs dt_args(PyObject *bias, PyObject *softplus, PyObject *limit, std::initializer_list<int64_t> bias_shape) {
  DtArgs d;
  const int sp = softplus == Py_True ? 1 : softplus == Py_False ? 0 : -1;
  if (sp < 0) return d;
  d.given = bias != Py_None || sp != 0 || limit != Py_None;
  if (bias != Py_None) {
    const Arg b = tensor(bias);
    if (!b.ok || !f32(b) || !is(b, bias_shape)) return d;
    d.x.dt_bias = static_cast<const float *>(b.ptr());
  }
  d.x.dt_softplus = sp;
  if (limit != Py_None) {
    if (!PyTuple_CheckExact(limit) || PyTuple_GET_SIZE(limit) != 2) return d;
    PyObject *lo = PyTuple_GET_ITEM(limit, 0), *hi = PyTuple_GET_ITEM(limit, 1);
    if (!PyFloat_CheckExact(lo) || !PyFloat_CheckExact(hi)) return d;
    d.x.dt_min = static_cast<float>(PyFloat_AS_DOUBLE(lo));
    d.x.dt_max = static_cast<float>(PyFloat_AS_DOUBLE(hi));
  }
  d.ok = true;
  return d;
}

// up to three widths that sum to the channel count; false: ask ssd.py
bool split_of(PyObject *split, int64_t channels, int32_t w[3]) {
  w[0] = static_cast<int32_t>(channels);
  w[1] = w[2] = 0;
  if (split == Py_None) return channels > 0;
  const bool tup = PyTuple_CheckExact(split);
  if (!tup && !PyList_CheckExact(split)) return false;
  const Py_ssize_t n = tup ? PyTuple_GET_SIZE(split) : PyList_GET_SIZE(split);
  if (n < 1 || n > 3) return false;
  int64_t sum = 0;
  w[0] = 0;
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject *o = tup ? PyTuple_GET_ITEM(split, i) : PyList_GET_ITEM(split, i);
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    if (over || v < 0 || v > INT32_MAX) return false;
    w[i] = static_cast<int32_t>(v);
    sum += v;
  }
  return sum == channels && w[0] >= 1;
}
int activation_of(PyObject *o) {
  if (!PyUnicode_CheckExact(o)) return -1;
  if (PyUnicode_CompareWithASCIIString(o, "silu") == 0) return 1;
  if (PyUnicode_CompareWithASCIIString(o, "none") == 0) return 0;
  return -1;
}

PyObject *none() { Py_RETURN_NONE; }
PyObject *failed(ssd_status st) { return PyLong_FromLong(st); }
PyObject *new_ref(PyObject *o) {
  Py_INCREF(o);
  return o;
}
template <typename F>
ssd_status released(F &&call) {  // (the call may wait for room in the stream's queue; nothing in it throws)
  ssd_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return st;
}
// The caller's output, or a new one like `like`: y is the reference that is returned.
bool output_like(PyObject *given, const Arg &like, at::Tensor &own, Arg &out) {
  if (given == Py_None) {
    own = at::empty_like(*like.t);
    out.t = &own;
    out.ok = true;
    return true;
  }
  out = tensor(given);
  return out.ok && out.t->scalar_type() == like.t->scalar_type() && out.t->numel() >= like.t->numel();
}
PyObject *result(PyObject *given, at::Tensor &own) { return given == Py_None ? THPVariable_Wrap(std::move(own)) : new_ref(given); }

#define SSD_ARGS(n) if (nargs != (n)) return none()

// (state, x, dt, A, B, C, D, y)
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  SSD_ARGS(8);
  const Arg state = tensor(a[0]), x = tensor(a[1]), dt = tensor(a[2]), A = tensor(a[3]), B = tensor(a[4]), C = tensor(a[5]), D = tensor(a[6]);
  if (!state.ok || !x.ok || !dt.ok || !A.ok || !B.ok || !C.ok || !D.ok || state.t->dim() != 4 || B.t->dim() != 3) return none();
  const int64_t Bt = state.t->size(0), H = state.t->size(1), P = state.t->size(2), N = state.t->size(3), G = B.t->size(1);
  const int io = io_of(x);
  if (io < 0 || !f32(state) || !f32(dt) || io_of(B) != io || io_of(C) != io || !f32_of(A, H) || !f32_of(D, H) ||
      !is(x, {Bt, H, P}) || !is(dt, {Bt, H}) || !is(B, {Bt, G, N}) || !is(C, {Bt, G, N}) || !fits({Bt, H, P, N, G}))
    return none();
  at::Tensor own;
  Arg y;
  if (!output_like(a[7], x, own, y)) return none();
  const ssd_shape sh = {(int32_t)Bt, 1, (int32_t)H, (int32_t)P, (int32_t)N, (int32_t)G, 1, io};
  void *const s = stream();
  float *const sp = (float *)state.ptr();
  const float *const dp = (const float *)dt.ptr(), *const Ap = (const float *)A.ptr(), *const Dp = (const float *)D.ptr();
  const void *const xp = x.ptr(), *const Bp = B.ptr(), *const Cp = C.ptr();
  void *const yp = y.ptr();
  const ssd_status st = released([&] { return api.decode_step(&sh, sp, xp, dp, Ap, Bp, Cp, Dp, yp, s); });
  return st != SSD_OK ? failed(st) : result(a[7], own);
  END_HANDLE_TH_ERRORS
}

// (state, x, dt, A, B, C, D, y, dt_bias, dt_softplus, dt_limit); steps: a leading axis of x, dt, B and C
template <bool kSteps>
PyObject *decode_layers(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  SSD_ARGS(11);
  constexpr int k = kSteps ? 1 : 0;
  const Arg state = tensor(a[0]), x = tensor(a[1]), dt = tensor(a[2]), A = tensor(a[3]), B = tensor(a[4]), C = tensor(a[5]), D = tensor(a[6]);
  if (!state.ok || !x.ok || !dt.ok || !A.ok || !B.ok || !C.ok || !D.ok || state.t->dim() != 5 || B.t->dim() != 4 + k || x.t->dim() != 4 + k)
    return none();
  const int64_t Ly = state.t->size(0), Bt = state.t->size(1), H = state.t->size(2), P = state.t->size(3), N = state.t->size(4), G = B.t->size(2 + k);
  const int64_t S = kSteps ? x.t->size(0) : 1;
  const int io = io_of(x);
  if (io < 0 || !f32(state) || !f32(dt) || !f32(A) || !f32(D) || io_of(B) != io || io_of(C) != io || !is(A, {Ly, H}) ||
      !is(D, {Ly, H}) || !fits({S, Ly, Bt, H, P, N, G}))
    return none();
  if (kSteps ? !is(x, {S, Ly, Bt, H, P}) || !is(dt, {S, Ly, Bt, H}) || !is(B, {S, Ly, Bt, G, N}) || !is(C, {S, Ly, Bt, G, N})
             : !is(x, {Ly, Bt, H, P}) || !is(dt, {Ly, Bt, H}) || !is(B, {Ly, Bt, G, N}) || !is(C, {Ly, Bt, G, N}))
    return none();
  const DtArgs xf = dt_args(a[8], a[9], a[10], {Ly, H});
  if (!xf.ok) return none();
  at::Tensor own;
  Arg y;
  if (!output_like(a[7], x, own, y)) return none();
  const ssd_shape sh = {(int32_t)Bt, 1, (int32_t)H, (int32_t)P, (int32_t)N, (int32_t)G, 1, io};
  void *const s = stream();
  float *const sp = (float *)state.ptr();
  const float *const dp = (const float *)dt.ptr(), *const Ap = (const float *)A.ptr(), *const Dp = (const float *)D.ptr();
  const void *const xp = x.ptr(), *const Bp = B.ptr(), *const Cp = C.ptr();
  void *const yp = y.ptr();
  const int32_t n = (int32_t)S, l = (int32_t)Ly;
  const ssd_status st = released([&] {
    if (kSteps)
      return xf.given ? api.decode_steps_dt(n, l, &sh, &xf.x, sp, xp, dp, Ap, Bp, Cp, Dp, yp, s)
                      : api.decode_steps(n, l, &sh, sp, xp, dp, Ap, Bp, Cp, Dp, yp, s);
    return xf.given ? api.decode_layers_dt(l, &sh, &xf.x, sp, xp, dp, Ap, Bp, Cp, Dp, yp, s)
                    : api.decode_layers(l, &sh, sp, xp, dp, Ap, Bp, Cp, Dp, yp, s);
  });
  return st != SSD_OK ? failed(st) : result(a[7], own);
  END_HANDLE_TH_ERRORS
}

// (x, dt, A, B, C, D, chunk, h0, y, final_state, workspace, dt_bias, dt_softplus, dt_limit); packed: cu_seqlens before chunk
template <bool kPacked>
PyObject *prefill(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  constexpr int k = kPacked ? 1 : 0;
  SSD_ARGS(14 + k);
  const Arg x = tensor(a[0]), dt = tensor(a[1]), A = tensor(a[2]), B = tensor(a[3]), C = tensor(a[4]), D = tensor(a[5]);
  const Arg cu = kPacked ? tensor(a[6]) : Arg(), h0 = tensor_or_none(a[7 + k]);
  PyObject *const gy = a[8 + k], *const gf = a[9 + k], *const gw = a[10 + k];
  if (!x.ok || !dt.ok || !A.ok || !B.ok || !C.ok || !D.ok || !h0.ok || x.t->dim() != 4 - k || B.t->dim() != 4 - k) return none();
  if (kPacked && (!cu.ok || cu.t->scalar_type() != at::kInt || cu.t->numel() < 2)) return none();
  const int64_t Bt = kPacked ? cu.t->numel() - 1 : x.t->size(0), T = x.t->size(1 - k), H = x.t->size(2 - k), P = x.t->size(3 - k);
  const int64_t G = B.t->size(2 - k), N = B.t->size(3 - k);
  int over = 0;
  if (!PyLong_CheckExact(a[6 + k])) return none();
  const long long chunk = PyLong_AsLongLongAndOverflow(a[6 + k], &over);
  const int io = io_of(x);
  if (over || io < 0 || !fits({Bt, T, H, P, N, G, chunk}) || io_of(B) != io || io_of(C) != io || !f32(dt) || !f32(A) || !f32(D) ||
      (h0.t != nullptr && (!f32(h0) || !is(h0, {Bt, H, P, N}))) || !is(A, {H}) || !is(D, {H}))
    return none();
  if (kPacked ? !is(dt, {T, H}) || !is(B, {T, G, N}) || !is(C, {T, G, N}) : !is(dt, {Bt, T, H}) || !is(B, {Bt, T, G, N}) || !is(C, {Bt, T, G, N}))
    return none();
  const DtArgs xf = dt_args(a[11 + k], a[12 + k], a[13 + k], {H});
  if (!xf.ok) return none();
  // (given ones are looked at before anything is allocated)
  at::Tensor own_y, own_f, own_w;
  Arg y, f, w;
  if (gy != Py_None && !output_like(gy, x, own_y, y)) return none();
  if (gf != Py_None && (!(f = tensor(gf)).ok || !f32_of(f, Bt * H * P * N))) return none();
  if (gw != Py_None && !(w = tensor(gw)).ok) return none();
  const ssd_shape sh = {(int32_t)Bt, (int32_t)T, (int32_t)H, (int32_t)P, (int32_t)N, (int32_t)G, (int32_t)chunk, io};
  if (gy == Py_None) output_like(gy, x, own_y, y);
  if (gf == Py_None) {
    own_f = at::empty({Bt, H, P, N}, x.t->options().dtype(at::kFloat));
    f.t = &own_f;
  }
  if (gw == Py_None) {
    const size_t need = kPacked ? api.varlen_workspace_bytes(&sh) : api.prefill_workspace_bytes(&sh);
    own_w = at::empty({(int64_t)(need > 256 ? need : 256)}, x.t->options().dtype(at::kByte));
    w.t = &own_w;
  }
  const size_t bytes = w.t->nbytes();
  void *const s = stream();
  const float *const dp = (const float *)dt.ptr(), *const Ap = (const float *)A.ptr(), *const Dp = (const float *)D.ptr();
  const float *const hp = (const float *)h0.ptr();
  float *const fp = (float *)f.ptr();
  const void *const xp = x.ptr(), *const Bp = B.ptr(), *const Cp = C.ptr();
  void *const yp = y.ptr(), *const wp = w.ptr();
  const int32_t *const cp = (const int32_t *)cu.ptr();
  const ssd_status st = released([&] {
    if (kPacked)
      return xf.given ? api.varlen_dt(&sh, &xf.x, cp, xp, dp, Ap, Bp, Cp, Dp, hp, yp, fp, wp, bytes, s)
                      : api.varlen(&sh, cp, xp, dp, Ap, Bp, Cp, Dp, hp, yp, fp, wp, bytes, s);
    return xf.given ? api.prefill_dt(&sh, &xf.x, xp, dp, Ap, Bp, Cp, Dp, hp, yp, fp, wp, bytes, s)
                    : api.prefill(&sh, xp, dp, Ap, Bp, Cp, Dp, hp, yp, fp, wp, bytes, s);
  });
  if (st != SSD_OK) return failed(st);
  PyObject *const ry = result(gy, own_y), *const rf = result(gf, own_f);
  PyObject *const both = ry != nullptr && rf != nullptr ? PyTuple_Pack(2, ry, rf) : nullptr;
  Py_XDECREF(ry);
  Py_XDECREF(rf);
  return both;
  END_HANDLE_TH_ERRORS
}

// prefill: (u, weight, bias, conv_state, split, activation); step: (conv_state, u, weight, bias, split, activation)
template <bool kStep>
PyObject *conv1d(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  SSD_ARGS(6);
  const Arg u = tensor(a[kStep ? 1 : 0]), weight = tensor(a[kStep ? 2 : 1]), bias = tensor_or_none(a[kStep ? 3 : 2]);
  const Arg state = kStep ? tensor(a[0]) : tensor_or_none(a[3]);
  const int act = activation_of(a[5]);
  if (!u.ok || !weight.ok || !bias.ok || !state.ok || act < 0 || u.t->dim() != (kStep ? 2 : 3) || weight.t->dim() != 2) return none();
  const int64_t Bt = u.t->size(0), T = kStep ? 1 : u.t->size(1), C = u.t->size(kStep ? 1 : 2), k = weight.t->size(1);
  const int io = io_of(u);
  int32_t w[3];
  if (io < 0 || !fits({Bt, T, C, k}) || k < 1 || !split_of(a[4], C, w) || !f32(weight) || !is(weight, {C, k}) ||
      (bias.t != nullptr && (!f32(bias) || !is(bias, {C}))) ||
      (state.t != nullptr && (state.t->scalar_type() != u.t->scalar_type() || !is(state, {Bt, C, k - 1}))))
    return none();
  at::Tensor out[3], new_state;
  void *z[3] = {nullptr, nullptr, nullptr};
  int n = 0;
  for (int i = 0; i < 3; ++i)
    if (w[i] > 0) {
      out[i] = kStep ? at::empty({Bt, w[i]}, u.t->options()) : at::empty({Bt, T, w[i]}, u.t->options());
      z[i] = out[i].data_ptr();
      ++n;
    }
  if (!kStep) new_state = at::empty({Bt, C, k - 1}, u.t->options());
  void *const s = stream(), *const sp = state.ptr(), *const np = kStep ? nullptr : new_state.data_ptr();
  const void *const up = u.ptr();
  const float *const Wp = (const float *)weight.ptr(), *const bp = (const float *)bias.ptr();
  const ssd_status st = released([&] {
    return kStep ? api.conv_step((int32_t)Bt, (int32_t)k, io, w, sp, up, Wp, bp, z[0], z[1], z[2], act, s)
                 : api.conv_prefill((int32_t)Bt, (int32_t)T, (int32_t)k, io, w, up, Wp, bp, sp, z[0], z[1], z[2], np, act, s);
  });
  if (st != SSD_OK) return failed(st);
  PyObject *const outs = PyList_New(n);
  if (outs == nullptr) return nullptr;
  for (int i = 0, at = 0; i < 3; ++i)
    if (w[i] > 0) PyList_SET_ITEM(outs, at++, THPVariable_Wrap(std::move(out[i])));
  if (kStep) return outs;
  PyObject *const rs = THPVariable_Wrap(std::move(new_state));
  PyObject *const both = PyTuple_Pack(2, outs, rs);
  Py_DECREF(outs);
  Py_DECREF(rs);
  return both;
  END_HANDLE_TH_ERRORS
}

// init(addresses): the functions of the C ABI in the order of Api
PyObject *init(PyObject *, PyObject *list) {
  constexpr Py_ssize_t kCount = sizeof(Api) / sizeof(void *);
  if (!PyList_Check(list) || PyList_GET_SIZE(list) != kCount) {
    PyErr_SetString(PyExc_ValueError, "a list of the addresses of the C ABI is expected");
    return nullptr;
  }
  void **const at = reinterpret_cast<void **>(&api);
  for (Py_ssize_t i = 0; i < kCount; ++i) {
    at[i] = PyLong_AsVoidPtr(PyList_GET_ITEM(list, i));
    if (at[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a function of the C ABI is missing");
      return nullptr;
    }
  }
  Py_RETURN_NONE;
}

#define SSD_FAST(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"init", init, METH_O, nullptr},
    SSD_FAST("decode_step", decode_step),
    SSD_FAST("decode_step_layers", decode_layers<false>),
    SSD_FAST("decode_steps_layers", decode_layers<true>),
    SSD_FAST("prefill", prefill<false>),
    SSD_FAST("prefill_varlen", prefill<true>),
    SSD_FAST("conv1d_prefill", conv1d<false>),
    SSD_FAST("conv1d_step", conv1d<true>),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ssd_binding", "Native marshalling of paper_2603_09555_amd.ssd, built for torch " SSD_TORCH_VERSION ";", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ssd_binding(void) {
  PyObject *const m = PyModule_Create(&module);
  // (torch's C++ interface has no stable binary form: ssd.py uses the module with the torch it was built for only)
  if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", SSD_TORCH_VERSION) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
