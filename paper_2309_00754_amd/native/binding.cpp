// The accepted form of the Python binding's calls, in native code: checks the
// tensors (dtype, device, contiguity, shape), takes their pointers and the
// current stream, and calls libhydra.  Whatever is not the accepted form (a
// host tensor, another dtype, a sequence that is no list or tuple, a missing
// workspace, a tensor subclass, an exception on the way) returns kSlow, and
// the Python function checks the arguments itself, with its own messages.
//
// Why: at decode sizes a call's host time is its time.  In Python, one
// condition of attribute reads per tensor and ctypes took 7.6 us for the small
// linear (its kernel 6.2), 19.8 for four projections (24 tensors; 15) and 7.5
// for each call of the PPO step (kernels 2.8 to 4.8).
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include "../../include/hydra.h"

namespace {

constexpr long kSlow = -1000;

enum Kind { kBf16, kF32, kI32, kU8 };

// Collects the arguments of one call; ok turns false at the first that is not
// of the accepted form.
struct Take {
  bool ok = true;

  const at::Tensor* tensor(PyObject* o, Kind kind) {
    if (!ok || o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) {
      ok = false;
      return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    const auto d = t.scalar_type();
    const bool dtype = kind == kBf16   ? d == at::kBFloat16 || d == at::kShort || d == at::kUInt16
                       : kind == kF32  ? d == at::kFloat
                       : kind == kI32  ? d == at::kInt
                                       : d == at::kByte;
    ok = t.is_cuda() && dtype && t.is_contiguous();
    return ok ? &t : nullptr;
  }
  // A matrix that has to be there: its sizes and pointer.
  const uint16_t* matrix(PyObject* o, int64_t& rows, int64_t& cols, Kind kind = kBf16) {
    const at::Tensor* t = tensor(o, kind);
    if (!t || t->dim() != 2) {
      ok = false;
      return nullptr;
    }
    rows = t->size(0);
    cols = t->size(1);
    return static_cast<const uint16_t*>(t->data_ptr());
  }
  int64_t rows(PyObject* o) {  // size(0) of a tensor, 0 for None
    if (!ok || o == Py_None) return 0;
    if (!THPVariable_CheckExact(o) || THPVariable_Unpack(o).dim() < 1) {
      ok = false;
      return 0;
    }
    return THPVariable_Unpack(o).size(0);
  }
  void* ptr(const at::Tensor* t, bool shape) {
    if (!ok || !t) return nullptr;
    if (!shape) {
      ok = false;
      return nullptr;
    }
    return t->data_ptr();
  }
  // None, or a tensor of this shape.
  template <class T>
  T* at1(PyObject* o, Kind kind, int64_t n) {
    const at::Tensor* t = tensor(o, kind);
    return static_cast<T*>(ptr(t, t && t->dim() == 1 && t->size(0) == n));
  }
  template <class T>
  T* at2(PyObject* o, Kind kind, int64_t n, int64_t m) {
    const at::Tensor* t = tensor(o, kind);
    return static_cast<T*>(ptr(t, t && t->dim() == 2 && t->size(0) == n && t->size(1) == m));
  }
  void* workspace(PyObject* o, size_t& bytes) {
    const at::Tensor* t = tensor(o, kU8);
    if (!t) {
      ok = false;
      return nullptr;
    }
    bytes = (size_t)t->numel();
    return t->data_ptr();
  }
  float real(PyObject* o) {
    if (!PyFloat_Check(o) && !PyLong_CheckExact(o)) {
      ok = false;
      return 0.f;
    }
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return (float)v;
  }
  int64_t whole(PyObject* o) {
    if (!PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    return v;
  }
  void* stream(PyObject* o) {
    if (!ok) return nullptr;
    if (o == Py_None) return reinterpret_cast<void*>(c10::hip::getCurrentHIPStream().stream());
    PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
    if (!h) {
      PyErr_Clear();
      ok = false;
      return nullptr;
    }
    void* p = PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
    if (PyErr_Occurred() || !PyLong_Check(h)) {
      PyErr_Clear();
      ok = false;
    }
    Py_DECREF(h);
    return p;
  }
  // n entries of a list or tuple; None (where allowed): n times None.
  PyObject* const* list(PyObject* o, int64_t n, bool may_be_none = false) {
    static PyObject* const nones[HYDRA_MAX_GROUP] = {Py_None, Py_None, Py_None, Py_None,
                                                     Py_None, Py_None, Py_None, Py_None};
    if (may_be_none && o == Py_None && n <= HYDRA_MAX_GROUP) return nones;
    if (!(PyList_CheckExact(o) || PyTuple_CheckExact(o)) || PySequence_Fast_GET_SIZE(o) != n) {
      ok = false;
      return nones;
    }
    return PySequence_Fast_ITEMS(o);
  }
};

// f(take) fills the arguments and returns the library call to make; the call
// itself runs without the interpreter's lock, as through ctypes.
template <class F>
PyObject* guarded(F&& f) {
  try {
    Take a;
    auto call = f(a);
    if (!a.ok) return PyLong_FromLong(kSlow);
    hydra_status st;
    Py_BEGIN_ALLOW_THREADS st = call();
    Py_END_ALLOW_THREADS return PyLong_FromLong((long)st);
  } catch (...) {
    PyErr_Clear();
    return PyLong_FromLong(kSlow);
  }
}

#define HYDRA_PY(name, count)                                                        \
  PyObject* name##_(PyObject* const* v);                                             \
  PyObject* name(PyObject*, PyObject* const* v, Py_ssize_t n) {                      \
    if (n != count) {                                                                \
      PyErr_SetString(PyExc_TypeError, #name ": wrong number of arguments");         \
      return nullptr;                                                                \
    }                                                                                \
    return name##_(v);                                                               \
  }                                                                                  \
  PyObject* name##_(PyObject* const* v)

// x W A B s y_off y_on workspace stream with_workspace
HYDRA_PY(lora_linear, 10) {
  return guarded([&](Take& a) {
    int64_t M = 0, K = 0, N = a.rows(v[1]), r = a.rows(v[2]);
    const uint16_t* x = a.matrix(v[0], M, K);
    const uint16_t* W = a.at2<uint16_t>(v[1], kBf16, N, K);
    const uint16_t* A = a.at2<uint16_t>(v[2], kBf16, r, K);
    const uint16_t* B = a.at2<uint16_t>(v[3], kBf16, N, r);
    const float s = a.real(v[4]);
    float* yo = a.at2<float>(v[5], kF32, M, N);
    float* yn = a.at2<float>(v[6], kF32, M, N);
    const bool with_ws = v[9] == Py_True;
    size_t bytes = 0;
    void* ws = with_ws ? a.workspace(v[7], bytes) : nullptr;
    a.ok = a.ok && W;
    void* st = a.stream(v[8]);
    return [=]() {
      return with_ws ? hydra_lora_linear_ws(x, W, A, B, s, M, N, K, r, yo, yn, ws, bytes, st)
                     : hydra_lora_linear(x, W, A, B, s, M, N, K, r, yo, yn, st);
    };
  });
}

// xs Ws As Bs ss y_offs y_ons workspace stream with_workspace
HYDRA_PY(lora_linear_group, 10) {
  struct Members {
    const uint16_t *x[HYDRA_MAX_GROUP], *W[HYDRA_MAX_GROUP], *A[HYDRA_MAX_GROUP], *B[HYDRA_MAX_GROUP];
    float *yo[HYDRA_MAX_GROUP], *yn[HYDRA_MAX_GROUP], s[HYDRA_MAX_GROUP];
  } m;
  return guarded([&](Take& a) {
    const int64_t G = PyList_CheckExact(v[1]) || PyTuple_CheckExact(v[1]) ? PySequence_Fast_GET_SIZE(v[1]) : 0;
    a.ok = G >= 1 && G <= HYDRA_MAX_GROUP;
    int64_t M = 0, K = 0, N = 0, r = 0;
    const bool with_ws = v[9] == Py_True;
    size_t bytes = 0;
    void* ws = nullptr;
    if (a.ok) {
      PyObject *const *xs = a.list(v[0], G), *const *Ws = a.list(v[1], G), *const *As = a.list(v[2], G),
                      *const *Bs = a.list(v[3], G), *const *ss = a.list(v[4], G),
                      *const *yo = a.list(v[5], G, true), *const *yn = a.list(v[6], G, true);
      if (a.ok) {
        a.matrix(xs[0], M, K);
        N = a.rows(Ws[0]);
        for (int64_t i = G - 1; i >= 0; --i)
          if (As[i] != Py_None) r = a.rows(As[i]);
        for (int64_t i = 0; i < G; ++i) {
          m.x[i] = a.at2<uint16_t>(xs[i], kBf16, M, K);
          m.W[i] = a.at2<uint16_t>(Ws[i], kBf16, N, K);
          m.A[i] = a.at2<uint16_t>(As[i], kBf16, r, K);
          m.B[i] = a.at2<uint16_t>(Bs[i], kBf16, N, r);
          m.yo[i] = a.at2<float>(yo[i], kF32, M, N);
          m.yn[i] = a.at2<float>(yn[i], kF32, M, N);
          m.s[i] = a.real(ss[i]);
        }
        if (with_ws) ws = a.workspace(v[7], bytes);
      }
    }
    void* st = a.stream(v[8]);
    return [=, &m]() {
      return with_ws ? hydra_lora_linear_group_ws(G, m.x, m.W, m.A, m.B, m.s, M, N, K, r, m.yo, m.yn, ws, bytes, st)
                     : hydra_lora_linear_group(G, m.x, m.W, m.A, m.B, m.s, M, N, K, r, m.yo, m.yn, st);
    };
  });
}

// x_off W x_ons As Bs ss y_off y_ons workspace stream with_workspace
HYDRA_PY(lora_linear_multi, 11) {
  struct Inputs {
    const uint16_t *x[HYDRA_MAX_ADAPTERS], *A[HYDRA_MAX_ADAPTERS], *B[HYDRA_MAX_ADAPTERS];
    float *yn[HYDRA_MAX_ADAPTERS], s[HYDRA_MAX_ADAPTERS];
  } m;
  return guarded([&](Take& a) {
    const int64_t n = PyList_CheckExact(v[2]) || PyTuple_CheckExact(v[2]) ? PySequence_Fast_GET_SIZE(v[2]) : -1;
    a.ok = n >= 1 && n <= HYDRA_MAX_ADAPTERS;
    int64_t M = 0, K = 0, N = 0, r = 0;
    const uint16_t *xo = nullptr, *W = nullptr;
    float* yo = nullptr;
    const bool with_ws = v[10] == Py_True;
    size_t bytes = 0;
    void* ws = nullptr;
    if (a.ok) {
      PyObject *const *xs = a.list(v[2], n), *const *As = a.list(v[3], n, true), *const *Bs = a.list(v[4], n, true),
                      *const *ss = a.list(v[5], n), *const *yn = a.list(v[7], n, true);
      if (a.ok) {
        a.matrix(v[0] != Py_None ? v[0] : xs[0], M, K);
        N = a.rows(v[1]);
        for (int64_t i = n - 1; i >= 0; --i)
          if (As[i] != Py_None) r = a.rows(As[i]);
        W = a.at2<uint16_t>(v[1], kBf16, N, K);
        xo = a.at2<uint16_t>(v[0], kBf16, M, K);
        yo = a.at2<float>(v[6], kF32, M, N);
        for (int64_t i = 0; i < n; ++i) {
          m.x[i] = a.at2<uint16_t>(xs[i], kBf16, M, K);
          m.A[i] = a.at2<uint16_t>(As[i], kBf16, r, K);
          m.B[i] = a.at2<uint16_t>(Bs[i], kBf16, N, r);
          m.yn[i] = a.at2<float>(yn[i], kF32, M, N);
          m.s[i] = a.real(ss[i]);
        }
        if (with_ws) ws = a.workspace(v[8], bytes);
      }
    }
    void* st = a.stream(v[9]);
    return [=, &m]() {
      return with_ws ? hydra_lora_linear_multi_ws(xo, W, n, m.x, m.A, m.B, m.s, M, N, K, r, yo, m.yn, ws, bytes, st)
                     : hydra_lora_linear_multi(xo, W, n, m.x, m.A, m.B, m.s, M, N, K, r, yo, m.yn, st);
    };
  });
}

// h_act h W_lm A B s tokens w_rm n_seq seq_len lp_on lp_off kl reward lse_on lse_off workspace err_flag stream
// own_scratch (h_act None: one input)
HYDRA_PY(score, 20) {
  return guarded([&](Take& a) {
    int64_t M = 0, K = 0, V = a.rows(v[2]), r = a.rows(v[3]);
    const uint16_t* h = a.matrix(v[1], M, K);
    const uint16_t* ha = a.at2<uint16_t>(v[0], kBf16, M, K);
    const uint16_t* W = a.at2<uint16_t>(v[2], kBf16, V, K);
    const uint16_t* A = a.at2<uint16_t>(v[3], kBf16, r, K);
    const uint16_t* B = a.at2<uint16_t>(v[4], kBf16, V, r);
    const float s = a.real(v[5]);
    const int32_t* tok = a.at1<int32_t>(v[6], kI32, M);
    const uint16_t* w_rm = a.at1<uint16_t>(v[7], kBf16, K);
    const int64_t n_seq = a.whole(v[8]), seq_len = a.whole(v[9]);
    float* lp_on = a.at1<float>(v[10], kF32, M);
    float* lp_off = a.at1<float>(v[11], kF32, M);
    float* kl = a.at1<float>(v[12], kF32, M);
    float* reward = a.at1<float>(v[13], kF32, n_seq);
    float* lse_on = a.at1<float>(v[14], kF32, M);
    float* lse_off = a.at1<float>(v[15], kF32, M);
    const bool own = v[19] == Py_True, two = v[0] != Py_None;
    size_t bytes = 0;
    void* ws = own ? nullptr : a.workspace(v[16], bytes);
    int32_t* err = a.at1<int32_t>(v[17], kI32, 1);
    a.ok = a.ok && W && n_seq >= 1 && seq_len >= 1 && n_seq <= M && seq_len <= M && n_seq * seq_len == M;
    void* st = a.stream(v[18]);
    return [=]() {
      if (own)
        return hydra_score_noalloc(h, W, A, B, s, tok, w_rm, n_seq, seq_len, K, V, r, lp_on, lp_off, kl, reward, lse_on,
                                   lse_off, err, st);
      if (two)
        return hydra_score_two_input(ha, h, W, A, B, s, tok, w_rm, n_seq, seq_len, K, V, r, lp_on, lp_off, kl, reward,
                                     lse_on, lse_off, ws, bytes, err, st);
      return hydra_score(h, W, A, B, s, tok, w_rm, n_seq, seq_len, K, V, r, lp_on, lp_off, kl, reward, lse_on, lse_off,
                         ws, bytes, err, st);
    };
  });
}

// logits_on logits_off tokens lp_on lp_off kl lse_on lse_off err_flag stream
HYDRA_PY(score_logits, 10) {
  return guarded([&](Take& a) {
    int64_t M = 0, V = 0;
    const void* on = a.matrix(v[0], M, V, kF32);
    const float* off = a.at2<float>(v[1], kF32, M, V);
    const int32_t* tok = a.at1<int32_t>(v[2], kI32, M);
    float* o[5];
    for (int i = 0; i < 5; ++i) o[i] = a.at1<float>(v[3 + i], kF32, M);
    int32_t* err = a.at1<int32_t>(v[8], kI32, 1);
    void* st = a.stream(v[9]);
    float *lp_on = o[0], *lp_off = o[1], *kl = o[2], *lse_on = o[3], *lse_off = o[4];
    return [=]() {
      return hydra_score_logits(static_cast<const float*>(on), off, tok, M, V, lp_on, lp_off, kl, lse_on, lse_off, err,
                                st);
    };
  });
}

// h w_v values stream
HYDRA_PY(value_head, 4) {
  return guarded([&](Take& a) {
    int64_t M = 0, K = 0;
    const uint16_t* h = a.matrix(v[0], M, K);
    const uint16_t* w = a.at1<uint16_t>(v[1], kBf16, K);
    float* values = a.at1<float>(v[2], kF32, M);
    void* st = a.stream(v[3]);
    return [=]() { return hydra_value_head(h, w, M, K, values, st); };
  });
}

// kl reward values n_seq seq_len start beta gamma lam rewards advantages returns stream
HYDRA_PY(ppo_advantages, 13) {
  return guarded([&](Take& a) {
    const int64_t n_seq = a.whole(v[3]), seq_len = a.whole(v[4]), start = a.whole(v[5]);
    a.ok = a.ok && n_seq >= 1 && seq_len >= 1 && n_seq <= (int64_t(1) << 40) / seq_len;
    const int64_t M = a.ok ? n_seq * seq_len : 0;
    const float* kl = a.at1<float>(v[0], kF32, M);
    const float* reward = a.at1<float>(v[1], kF32, n_seq);
    const float* values = a.at1<float>(v[2], kF32, M);
    const float beta = a.real(v[6]), gamma = a.real(v[7]), lam = a.real(v[8]);
    float* rewards = a.at1<float>(v[9], kF32, M);
    float* adv = a.at1<float>(v[10], kF32, M);
    float* ret = a.at1<float>(v[11], kF32, M);
    void* st = a.stream(v[12]);
    return [=]() {
      return hydra_ppo_advantages(kl, reward, values, n_seq, seq_len, start, beta, gamma, lam, rewards, adv, ret, st);
    };
  });
}

// lp_new lp_old advantages values returns n_seq seq_len start eps losses d_lp d_v stream
HYDRA_PY(ppo_loss, 13) {
  return guarded([&](Take& a) {
    const int64_t n_seq = a.whole(v[5]), seq_len = a.whole(v[6]), start = a.whole(v[7]);
    a.ok = a.ok && n_seq >= 1 && seq_len >= 1 && n_seq <= (int64_t(1) << 40) / seq_len;
    const int64_t M = a.ok ? n_seq * seq_len : 0;
    const float* in[5];
    for (int i = 0; i < 5; ++i) in[i] = a.at1<float>(v[i], kF32, M);
    const float eps = a.real(v[8]);
    float* losses = a.at1<float>(v[9], kF32, 3);
    float* d_lp = a.at1<float>(v[10], kF32, M);
    float* d_v = a.at1<float>(v[11], kF32, M);
    void* st = a.stream(v[12]);
    const float *lp_new = in[0], *lp_old = in[1], *adv = in[2], *values = in[3], *returns = in[4];
    return [=]() {
      return hydra_ppo_loss(lp_new, lp_old, adv, values, returns, n_seq, seq_len, start, eps, losses, d_lp, d_v, st);
    };
  });
}

// x Wt A B s dy dx dA dB workspace stream
HYDRA_PY(lora_linear_backward, 11) {
  return guarded([&](Take& a) {
    int64_t M = 0, N = 0, r = 0, K = 0;
    const uint16_t* dy = a.matrix(v[5], M, N);
    const uint16_t* A = a.matrix(v[2], r, K);  // (without an adapter: the Python path)
    const uint16_t* x = a.at2<uint16_t>(v[0], kBf16, M, K);
    const uint16_t* Wt = a.at2<uint16_t>(v[1], kBf16, K, N);
    const uint16_t* B = a.at2<uint16_t>(v[3], kBf16, N, r);
    const float s = a.real(v[4]);
    float* dx = a.at2<float>(v[6], kF32, M, K);
    float* dA = a.at2<float>(v[7], kF32, r, K);
    float* dB = a.at2<float>(v[8], kF32, N, r);
    size_t bytes = 0;
    void* ws = a.workspace(v[9], bytes);
    void* st = a.stream(v[10]);
    return [=]() { return hydra_lora_linear_backward(x, Wt, A, B, s, dy, M, N, K, r, dx, dA, dB, ws, bytes, st); };
  });
}

#define HYDRA_DEF(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HYDRA_DEF(lora_linear),  HYDRA_DEF(lora_linear_group), HYDRA_DEF(lora_linear_multi),
                         HYDRA_DEF(score),        HYDRA_DEF(score_logits),      HYDRA_DEF(value_head),
                         HYDRA_DEF(ppo_advantages), HYDRA_DEF(ppo_loss),        HYDRA_DEF(lora_linear_backward),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hydra_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__hydra_native() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddIntConstant(m, "SLOW", kSlow) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
