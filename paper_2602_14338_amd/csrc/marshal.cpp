// The binding's native part.
//
//   group_advantage(...), logprob_fwd(...), ...: a whole call whose arguments are all plain - tensors of the expected dtype,
//   on the GPU and contiguous, ints that fit, floats - straight to the entry point whose address bind() was given.
//   Anything else, also whatever the call would refuse, gives NotImplemented with nothing done, and the binding goes
//   its general way, which converts or raises.  (ctypes and the parameter structure were 2 of the 5.7 us of a call that
//   launches one small kernel.)
//
// Checks and device pointers of a call's tensors in one step: the part of the binding that costs most of a small
// call when it runs in Python (fifteen tensors at 0.5 us each against 3 us for a launch).
//
//   pointers(t0, dtype0, name0, t1, dtype1, name1, ...) -> (address or None, ...)
//
// Per tensor, in this order: None stays None; it must live on the GPU, have the dtype (None: any) and be
// contiguous.  Anything but a plain tensor or parameter goes to the Python function given to setup(), which
// performs the same checks.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include "../../include/aero.h"

namespace {

PyObject* g_error = nullptr;      // exception class of the binding
PyObject* g_general = nullptr;    // pointer of any other kind of tensor: f(t, dtype, name)

PyObject* setup(PyObject*, PyObject* args) {
  PyObject *error, *general;
  if (!PyArg_ParseTuple(args, "OO", &error, &general)) return nullptr;
  Py_INCREF(error);
  Py_INCREF(general);
  Py_XSETREF(g_error, error);
  Py_XSETREF(g_general, general);
  Py_RETURN_NONE;
}

PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (!g_error || n_args % 3 != 0) {
    PyErr_SetString(PyExc_TypeError, "pointers: expected (tensor, dtype, name) triples after setup()");
    return nullptr;
  }
  THPObjectPtr out(PyTuple_New(n_args / 3));
  if (!out) return nullptr;
  for (Py_ssize_t i = 0; i < n_args; i += 3) {
    PyObject *t = args[i], *dtype = args[i + 1], *name = args[i + 2], *value;
    if (t == Py_None) {
      value = Py_NewRef(Py_None);
    } else if (!THPVariable_CheckExact(t)) {
      value = PyObject_CallFunctionObjArgs(g_general, t, dtype, name, nullptr);
    } else {
      const at::Tensor& x = THPVariable_Unpack(t);
      if (!x.is_cuda()) {
        PyErr_Format(g_error, "%U: expected a GPU tensor", name);
        return nullptr;
      }
      if (dtype != Py_None && x.scalar_type() != reinterpret_cast<THPDtype*>(dtype)->scalar_type) {
        THPObjectPtr got(PyObject_GetAttrString(t, "dtype"));
        if (got) PyErr_Format(g_error, "%U: expected dtype %S, got %S", name, dtype, got.get());
        return nullptr;
      }
      if (!x.is_contiguous()) {
        PyErr_Format(g_error, "%U: expected a contiguous tensor", name);
        return nullptr;
      }
      value = PyLong_FromVoidPtr(x.data_ptr());
    }
    if (!value) return nullptr;
    PyTuple_SET_ITEM(out.get(), i / 3, value);
  }
  return out.release();
  END_HANDLE_TH_ERRORS
}

// ---- whole calls ----
PyObject* g_stream = nullptr;     // torch's current raw stream of a device index
PyObject* g_params = nullptr;     // class of group_advantage's parameters
decltype(&aero_group_advantage) g_group_advantage = nullptr;
decltype(&aero_logprob_fwd) g_logprob_fwd = nullptr;
decltype(&aero_grpo_loss_bwd) g_loss_bwd = nullptr;
decltype(&aero_grpo_loss_bwd_noalloc) g_loss_bwd_noalloc = nullptr;
decltype(&aero_lmhead_logprob_fused) g_fused = nullptr;

PyObject* bind(PyObject*, PyObject* args) {
  PyObject *stream, *params;
  unsigned long long f[5];
  if (!PyArg_ParseTuple(args, "OOKKKKK", &stream, &params, &f[0], &f[1], &f[2], &f[3], &f[4])) return nullptr;
  Py_INCREF(stream);
  Py_INCREF(params);
  Py_XSETREF(g_stream, stream);
  Py_XSETREF(g_params, params);
  g_group_advantage = reinterpret_cast<decltype(g_group_advantage)>(f[0]);
  g_logprob_fwd = reinterpret_cast<decltype(g_logprob_fwd)>(f[1]);
  g_loss_bwd = reinterpret_cast<decltype(g_loss_bwd)>(f[2]);
  g_loss_bwd_noalloc = reinterpret_cast<decltype(g_loss_bwd_noalloc)>(f[3]);
  g_fused = reinterpret_cast<decltype(g_fused)>(f[4]);
  Py_RETURN_NONE;
}

// The arguments of a call, taken in order; ok turns false at the first one that is not plain.
struct Plain {
  PyObject* const* next;
  bool ok = true;

  const at::Tensor* tensor() {   // nullptr: None, or not plain
    PyObject* o = *next++;
    if (o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) {
      ok = false;
      return nullptr;
    }
    const at::Tensor& x = THPVariable_Unpack(o);
    if (!x.is_cuda() || !x.is_contiguous()) ok = false;
    return &x;
  }
  void* any() {
    const at::Tensor* x = tensor();
    return x && ok ? x->data_ptr() : nullptr;
  }
  template <class T> T* of(at::ScalarType type) {
    const at::Tensor* x = tensor();
    if (x && x->scalar_type() != type) ok = false;
    return x && ok ? static_cast<T*>(x->data_ptr()) : nullptr;
  }
  float* f32() { return of<float>(at::kFloat); }
  int32_t* i32() { return of<int32_t>(at::kInt); }
  uint8_t* u8() { return of<uint8_t>(at::kByte); }
  int64_t integer(int64_t lo, int64_t hi) { return integer_of(*next++, lo, hi); }
  int64_t integer_of(PyObject* o, int64_t lo, int64_t hi) {
    int overflow = 1;
    const int64_t v = PyLong_CheckExact(o) ? PyLong_AsLongLongAndOverflow(o, &overflow) : 0;
    if (overflow || v < lo || v > hi) ok = false;
    return v;
  }
  int32_t int32() { return int32_t(integer(INT32_MIN, INT32_MAX)); }
  int64_t int64() { return integer(INT64_MIN, INT64_MAX); }
  float real() { return real_of(*next++); }
  float real_of(PyObject* o) {
    if (PyFloat_CheckExact(o)) return float(PyFloat_AS_DOUBLE(o));
    return float(integer_of(o, -(1 << 24), 1 << 24));
  }
};

// Storage code of logits (-1: none).
int32_t dtype_code(const at::Tensor& x) {
  switch (x.scalar_type()) {
    case at::kFloat: return AERO_F32;
    case at::kBFloat16: return AERO_BF16;
    case at::kHalf: return AERO_F16;
    case at::kFloat8_e4m3fn: return AERO_F8E4M3;
    default: return -1;
  }
}

// torch's current stream on the tensor's device.
bool stream_of(const at::Tensor& x, void** stream) {
  THPObjectPtr device(PyLong_FromLong(x.get_device()));
  if (!device) return false;
  THPObjectPtr handle(PyObject_CallOneArg(g_stream, device));
  if (!handle) return false;
  *stream = PyLong_AsVoidPtr(handle);
  return !PyErr_Occurred();
}

// A call whose arguments are plain: the entry point without the interpreter lock, its status as an int.
template <class Call> PyObject* finish(const Plain& p, const at::Tensor* on, Call call) {
  if (!p.ok || !on) Py_RETURN_NOTIMPLEMENTED;
  void* stream = nullptr;
  if (!stream_of(*on, &stream)) return nullptr;
  aero_status status;
  Py_BEGIN_ALLOW_THREADS
  status = call(stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

const at::Tensor* peek(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

PyObject* group_advantage(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 15 || !g_group_advantage) Py_RETURN_NOTIMPLEMENTED;
  static PyObject* names[9];
  if (!names[8]) {
    const char* const text[9] = {"k_ratio", "s_rescue", "tau_num", "tau_den", "zero_keep", "reject_enable", "posterior_mode", "alpha0", "beta0"};
    for (int k = 0; k < 9; ++k)
      if (!(names[k] = PyUnicode_InternFromString(text[k]))) return nullptr;
  }
  Plain p{args};
  const float* rewards = p.f32();
  const int32_t* lengths = p.i32();
  const at::Tensor* on = peek(*p.next);
  const int32_t* offsets = p.i32();
  const uint32_t* keys = static_cast<uint32_t*>(p.any());
  const int32_t Q = p.int32(), R = p.int32();
  PyObject* params = *p.next++;
  if (reinterpret_cast<PyObject*>(Py_TYPE(params)) != g_params) Py_RETURN_NOTIMPLEMENTED;
  int32_t whole[7];
  float prior[2];
  for (int k = 0; k < 9; ++k) {
    THPObjectPtr v(PyObject_GetAttr(params, names[k]));
    if (!v) {   // no such attribute: the general way raises
      PyErr_Clear();
      Py_RETURN_NOTIMPLEMENTED;
    }
    if (k < 7) whole[k] = int32_t(p.integer_of(v, INT32_MIN, INT32_MAX));
    else prior[k - 7] = p.real_of(v);
  }
  const aero_adv_params c{whole[0], whole[1], whole[2], whole[3], whole[4], whole[5], whole[6], prior[0], prior[1]};
  float *adv = p.f32(), *weight = p.f32();
  uint8_t* mask = p.u8();
  int32_t *index = p.i32(), *kept = p.i32();
  uint8_t *zero_var = p.u8(), *category = p.u8();
  int32_t* err = p.i32();
  return finish(p, on, [&](void* s) {
    return g_group_advantage(rewards, lengths, offsets, keys, Q, R, &c, adv, weight, mask, index, kept, zero_var, category, err, s);
  });
  END_HANDLE_TH_ERRORS
}

PyObject* logprob_fwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 10 || !g_logprob_fwd) Py_RETURN_NOTIMPLEMENTED;
  Plain p{args};
  const at::Tensor* on = peek(*p.next);
  const void* logits = p.any();
  const int32_t dtype = on ? dtype_code(*on) : -1;
  if (dtype < 0) p.ok = false;
  const int64_t T = p.int64();
  const int32_t V = p.int32();
  const int64_t ld = p.int64();
  const int32_t* targets = p.i32();
  const uint8_t* active = p.u8();
  float *logprob = p.f32(), *entropy = p.f32(), *lse = p.f32();
  int32_t* err = p.i32();
  return finish(p, on, [&](void* s) { return g_logprob_fwd(logits, dtype, T, V, ld, targets, active, logprob, entropy, lse, err, s); });
  END_HANDLE_TH_ERRORS
}

// loss_bwd(logits, T, V, ld, targets, lse, entropy, old_logprob, token_rollout, adv, weight, R, eps_lo, eps_hi, grad_scale,
//          entropy_coef, kl_coef, ref_logprob, loss, clip_frac, logprob_out, entropy_out, lse_out, dlogits, err_flag
//          [, workspace]): with the workspace aero_grpo_loss_bwd, without it aero_grpo_loss_bwd_noalloc
PyObject* loss_bwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if ((n != 25 && n != 26) || !g_loss_bwd) Py_RETURN_NOTIMPLEMENTED;
  Plain p{args};
  const at::Tensor* on = peek(*p.next);
  const void* logits = p.any();
  const int32_t dtype = on ? dtype_code(*on) : -1;
  if (dtype < 0) p.ok = false;
  const int64_t T = p.int64();
  const int32_t V = p.int32();
  const int64_t ld = p.int64();
  const int32_t* targets = p.i32();
  const float *lse = p.f32(), *entropy = p.f32(), *old = p.f32();
  const int32_t* owner = p.i32();
  const float *adv = p.f32(), *weight = p.f32();
  const int32_t R = p.int32();
  const float eps_lo = p.real(), eps_hi = p.real(), scale = p.real(), ent_coef = p.real(), kl_coef = p.real();
  const float* ref = p.f32();
  float *loss = p.f32(), *clip = p.f32(), *lp_out = p.f32(), *ent_out = p.f32(), *lse_out = p.f32();
  const at::Tensor* d = peek(*p.next);
  void* dlogits = p.any();
  if (d && on && d->scalar_type() != on->scalar_type()) p.ok = false;
  int32_t* err = p.i32();
  if (n == 25)
    return finish(p, on, [&](void* s) {
      return g_loss_bwd_noalloc(logits, dtype, T, V, ld, targets, lse, entropy, old, owner, adv, weight, R, eps_lo, eps_hi, scale,
                                ent_coef, kl_coef, ref, loss, clip, lp_out, ent_out, lse_out, dlogits, err, s);
    });
  const at::Tensor* w = peek(*p.next);
  void* ws = p.any();
  const size_t bytes = w ? w->nbytes() : 0;
  return finish(p, on, [&](void* s) {
    return g_loss_bwd(logits, dtype, T, V, ld, targets, lse, entropy, old, owner, adv, weight, R, eps_lo, eps_hi, scale, ent_coef,
                      kl_coef, ref, loss, clip, lp_out, ent_out, lse_out, dlogits, err, ws, bytes, s);
  });
  END_HANDLE_TH_ERRORS
}

// fused(hidden, weight, T, H, V, targets, logprob, entropy, lse, old_logprob, token_rollout, adv, weight_rollout, R, eps_lo,
//       eps_hi, grad_scale, entropy_coef, kl_coef, ref_logprob, loss, clip_frac, dhidden, dweight, dweight_accumulate, err_flag,
//       workspace)
PyObject* fused(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 27 || !g_fused) Py_RETURN_NOTIMPLEMENTED;
  Plain p{args};
  const at::Tensor* on = peek(*p.next);
  const void *hidden = p.of<void>(at::kBFloat16), *weight = p.of<void>(at::kBFloat16);
  const int64_t T = p.int64();
  const int32_t H = p.int32(), V = p.int32();
  const int32_t* targets = p.i32();
  float *logprob = p.f32(), *entropy = p.f32(), *lse = p.f32();
  const float* old = p.f32();
  const int32_t* owner = p.i32();
  const float *adv = p.f32(), *weight_rollout = p.f32();
  const int32_t R = p.int32();
  const float eps_lo = p.real(), eps_hi = p.real(), scale = p.real(), ent_coef = p.real(), kl_coef = p.real();
  const float* ref = p.f32();
  float *loss = p.f32(), *clip = p.f32();
  void* dhidden = p.of<void>(at::kBFloat16);
  const at::Tensor* dw = peek(*p.next);
  void* dweight = p.any();
  int32_t dw_dtype = dw ? dtype_code(*dw) : AERO_F32;
  if (dw_dtype < 0) p.ok = false;
  PyObject* accumulate = *p.next++;
  if (accumulate == Py_True) dw_dtype |= AERO_DW_ACCUMULATE;
  else if (accumulate != Py_False) p.ok = false;
  int32_t* err = p.i32();
  const at::Tensor* w = peek(*p.next);
  void* ws = p.any();
  const size_t bytes = w ? w->nbytes() : 0;
  return finish(p, on, [&](void* s) {
    return g_fused(hidden, weight, T, H, V, targets, logprob, entropy, lse, old, owner, adv, weight_rollout, R, eps_lo, eps_hi, scale,
                   ent_coef, kl_coef, ref, loss, clip, dhidden, dweight, dw_dtype, err, ws, bytes, s);
  });
  END_HANDLE_TH_ERRORS
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)> constexpr PyCFunction fast() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F));
}

PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, "setup(error class, pointer function for other kinds of tensors)"},
    {"bind", bind, METH_VARARGS, "bind(raw stream function, parameter class, five entry points' addresses)"},
    {"pointers", fast<pointers>(), METH_FASTCALL, "pointers(t0, dtype0, name0, ...) -> tuple of addresses"},
    {"group_advantage", fast<group_advantage>(), METH_FASTCALL, "status, or NotImplemented"},
    {"logprob_fwd", fast<logprob_fwd>(), METH_FASTCALL, "status, or NotImplemented"},
    {"loss_bwd", fast<loss_bwd>(), METH_FASTCALL, "status, or NotImplemented"},
    {"fused", fast<fused>(), METH_FASTCALL, "status, or NotImplemented"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
