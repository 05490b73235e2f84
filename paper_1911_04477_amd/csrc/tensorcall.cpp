// The entry points of bnn.h that a program calls once per layer, taken straight from torch tensors.
//
// A layer on a few thousand values is a launch of 2.4 us, and checking and converting its tensors through Python's attribute
// calls (about 50 ns each, 20 to 30 of them) was 1.6 to 2 us beside it.  Here it is 0.2: one call from the binding with the
// tensors themselves.  Each function returns the status of the call, or None for anything but the plain case (tensors of
// the binding's types on the GPU, given outputs, integers, pairs of integers); the binding's own code then takes the call,
// and raises what it raises.  bind(): addresses of the library's functions, in the order of `names`.  built_for: the torch and the
// Python of whose objects this file's accessors know the layout; the binding uses it with no other.
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstring>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

#include "bnn.h"

namespace {

struct Library {
  decltype(&bnn_xnor_gemm) gemm;
  decltype(&bnn_xnor_gemm_epilogue) epilogue;
  decltype(&bnn_encode) encode;
  decltype(&bnn_conv2d) conv2d;
  decltype(&bnn_conv2d_packed) conv2d_packed;
  decltype(&bnn_im2col_packed) im2col;
  decltype(&bnn_conv2d_f32_sign) f32_sign;
  decltype(&bnn_conv2d_f32) f32;
  decltype(&bnn_maxpool2x2) maxpool;
  decltype(&bnn_fc_f32) fc;
};
constexpr const char *names[] = {"bnn_xnor_gemm", "bnn_xnor_gemm_epilogue", "bnn_encode", "bnn_conv2d", "bnn_conv2d_packed",
                                 "bnn_im2col_packed", "bnn_conv2d_f32_sign", "bnn_conv2d_f32", "bnn_maxpool2x2", "bnn_fc_f32"};
Library lib = {};

struct Other {};  // not the plain case

// The arguments of a call, taken in order.
class Args {
 public:
  Args(PyObject *const *a, Py_ssize_t n, Py_ssize_t want) : a_(a) {
    // subclasses and modes may give a tensor's attributes another meaning
    if (n != want || !lib.gemm || at::impl::torch_function_mode_enabled()) throw Other();
  }
  const at::Tensor &tensor() {
    PyObject *o = *a_++;
    if (!THPVariable_CheckExact(o)) throw Other();
    return THPVariable_Unpack(o);
  }
  const at::Tensor &tensor(at::ScalarType type) {
    const at::Tensor &t = tensor();
    if (!t.is_cuda() || t.scalar_type() != type) throw Other();
    return t;
  }
  const at::Tensor &tensor(at::ScalarType type, int64_t dim) {
    const at::Tensor &t = tensor(type);
    if (t.dim() != dim) throw Other();
    return t;
  }
  void *pointer() {  // of any tensor, or None
    if (*a_ == Py_None) {
      ++a_;
      return nullptr;
    }
    return tensor().data_ptr();
  }
  int64_t integer() { return integer(*a_++); }
  int small() { return as_int(integer()); }
  void pair(int (&v)[2]) {
    PyObject *o = *a_++;
    if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 2) throw Other();
    for (int i = 0; i < 2; ++i) v[i] = as_int(integer(PyTuple_GET_ITEM(o, i)));
  }

 private:
  static int64_t integer(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw Other();
    int overflow;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) throw Other();
    return v;
  }
  static int as_int(int64_t v) {
    if (v != (int)v) throw Other();
    return (int)v;
  }
  PyObject *const *a_;
};

int size(const at::Tensor &t, int64_t d) {
  const int64_t n = t.size(d);
  if (n != (int)n) throw Other();
  return (int)n;
}

float *f32(void *p) { return static_cast<float *>(p); }
int32_t *i32(void *p) { return static_cast<int32_t *>(p); }
uint64_t *u64(const at::Tensor &t) { return static_cast<uint64_t *>(t.data_ptr()); }
// rows of a matrix: one row may have any stride
int64_t row_stride(const at::Tensor &t, int64_t least) { return t.size(0) > 1 ? t.stride(0) : least; }

// Other threads run meanwhile; held again also where the call throws.
struct Released {
  PyThreadState *state = PyEval_SaveThread();
  ~Released() { PyEval_RestoreThread(state); }
};

template <class Call>
PyObject *launch(const Call &call) {
  void *const stream = c10::hip::getCurrentHIPStream().stream();
  bnn_status st;
  {
    Released released;
    st = call(stream);
  }
  return PyLong_FromLong((long)st);
}

// body(args) -> PyObject *; whatever it throws: not the plain case (tensors without storage throw c10::Error).
template <class Body>
PyObject *guarded(PyObject *const *a, Py_ssize_t n, Py_ssize_t want, const Body &body) {
  try {
    Args args(a, n, want);
    return body(args);
  } catch (...) {
    Py_RETURN_NONE;
  }
}

using at::kFloat;
using at::kInt;
using at::kLong;

PyObject *gemm(PyObject *, PyObject *const *a, Py_ssize_t n) {  // A, B, K, C
  return guarded(a, n, 4, [](Args &v) {
    const at::Tensor &A = v.tensor(kLong, 2), &B = v.tensor(kLong, 2);
    const int64_t K = v.integer();
    const at::Tensor &C = v.tensor(kInt, 2);
    const int64_t M = A.size(0), N = B.size(0), lda = row_stride(A, std::max<int64_t>(A.size(1), 1)),
                  ldb = row_stride(B, std::max<int64_t>(B.size(1), 1)), ldc = M > 1 ? C.stride(0) : std::max<int64_t>(N, 1);
    const uint64_t *const pa = u64(A), *const pb = u64(B);
    int32_t *const pc = i32(C.data_ptr());
    return launch([&](void *s) { return lib.gemm(pa, lda, pb, ldb, pc, ldc, M, N, K, s); });
  });
}

PyObject *epilogue(PyObject *, PyObject *const *a, Py_ssize_t n) {  // A, B, K, scale, bias, axis, Y
  return guarded(a, n, 7, [](Args &v) {
    const at::Tensor &A = v.tensor(kLong, 2), &B = v.tensor(kLong, 2);
    const int64_t K = v.integer();
    const float *const sc = f32(v.pointer()), *const bi = f32(v.pointer());
    const int axis = v.small();
    const at::Tensor &Y = v.tensor(kFloat, 2);
    const int64_t M = A.size(0), N = B.size(0), lda = row_stride(A, std::max<int64_t>(A.size(1), 1)),
                  ldb = row_stride(B, std::max<int64_t>(B.size(1), 1)), ld = std::max<int64_t>(N, 1);
    if (Y.size(0) != M || Y.size(1) != N || !Y.is_contiguous()) throw Other();
    const uint64_t *const pa = u64(A), *const pb = u64(B);
    float *const py = f32(Y.data_ptr());
    return launch([&](void *s) { return lib.epilogue(pa, lda, pb, ldb, M, N, K, nullptr, ld, py, ld, sc, bi, (bnn_ch_axis)axis, s); });
  });
}

PyObject *encode(PyObject *, PyObject *const *a, Py_ssize_t n) {  // src, dst
  return guarded(a, n, 2, [](Args &v) {
    const at::Tensor &src = v.tensor(kFloat, 2), &dst = v.tensor(kLong, 2);
    if (src.stride(1) != 1 || dst.stride(1) != 1) throw Other();
    const int64_t rows = src.size(0), K = src.size(1), Kw = K / 64 + (K % 64 != 0);
    const int64_t ls = rows > 1 ? src.stride(0) : std::max(K, src.stride(0)), ld = rows > 1 ? dst.stride(0) : std::max(Kw, dst.stride(0));
    const float *const ps = f32(src.data_ptr());
    uint64_t *const pd = u64(dst);
    return launch([&](void *s) { return lib.encode(ps, rows, K, ls, pd, ld, s); });
  });
}

PyObject *conv2d(PyObject *, PyObject *const *a, Py_ssize_t n) {  // x, w, D, kH, kW, stride, pad, out_i32, out_f32, scale, bias, workspace
  return guarded(a, n, 12, [](Args &v) {
    const at::Tensor &x = v.tensor(kFloat, 4), &w = v.tensor(kLong);
    const int D = v.small(), kH = v.small(), kW = v.small();
    int st[2], pd[2];
    v.pair(st);
    v.pair(pd);
    int32_t *const oi = i32(v.pointer());
    float *const of = f32(v.pointer());
    const float *const sc = f32(v.pointer()), *const bi = f32(v.pointer());
    const at::Tensor &ws = v.tensor();
    if (!x.is_contiguous() || !w.is_contiguous()) throw Other();
    const int N = size(x, 0), C = size(x, 1), H = size(x, 2), W = size(x, 3);
    const float *const px = f32(x.data_ptr());
    const uint64_t *const pw = u64(w);
    void *const pws = ws.data_ptr();
    const size_t nws = (size_t)ws.numel();
    return launch([&](void *s) {
      return lib.conv2d(px, pw, N, C, H, W, D, kH, kW, st[0], st[1], pd[0], pd[1], oi, of, sc, bi, pws, nws, s);
    });
  });
}

PyObject *conv2d_packed(PyObject *, PyObject *const *a, Py_ssize_t n) {  // xp, w, C, D, kH, kW, stride, pad, pool, i32, f32, packed, scale, bias
  return guarded(a, n, 14, [](Args &v) {
    const at::Tensor &x = v.tensor(kLong, 4), &w = v.tensor(kLong);
    const int C = v.small(), D = v.small(), kH = v.small(), kW = v.small();
    int st[2], pd[2];
    v.pair(st);
    v.pair(pd);
    const int pool = v.small();
    int32_t *const oi = i32(v.pointer());
    float *const of = f32(v.pointer());
    uint64_t *const op = static_cast<uint64_t *>(v.pointer());
    const float *const sc = f32(v.pointer()), *const bi = f32(v.pointer());
    if (!x.is_contiguous() || !w.is_contiguous() || C <= 0 || x.size(3) != ((int64_t)C + 63) / 64) throw Other();
    const int N = size(x, 0), H = size(x, 1), W = size(x, 2);
    const uint64_t *const px = u64(x), *const pw = u64(w);
    return launch([&](void *s) {
      return lib.conv2d_packed(px, pw, N, C, H, W, D, kH, kW, st[0], st[1], pd[0], pd[1], pool, oi, of, op, sc, bi, s);
    });
  });
}

PyObject *im2col(PyObject *, PyObject *const *a, Py_ssize_t n) {  // x, kH, kW, stride, pad, cols, workspace
  return guarded(a, n, 7, [](Args &v) {
    const at::Tensor &x = v.tensor(kFloat, 4);
    const int kH = v.small(), kW = v.small();
    int st[2], pd[2];
    v.pair(st);
    v.pair(pd);
    const at::Tensor &cols = v.tensor(kLong), &ws = v.tensor();
    if (!x.is_contiguous() || !cols.is_contiguous()) throw Other();
    const int N = size(x, 0), C = size(x, 1), H = size(x, 2), W = size(x, 3);
    // what the binding requires of cols, where its own arithmetic is plain
    if (kH <= 0 || kW <= 0 || st[0] <= 0 || st[1] <= 0 || pd[0] < 0 || pd[1] < 0) throw Other();
    const int64_t h = (int64_t)H + 2 * (int64_t)pd[0] - kH, w = (int64_t)W + 2 * (int64_t)pd[1] - kW;
    if (h < 0 || w < 0 || (double)N * (h / st[0] + 1) * (w / st[1] + 1) * kH * kW * (C / 64 + 1) > 1e15) throw Other();
    if (cols.numel() != N * (h / st[0] + 1) * (w / st[1] + 1) * kH * kW * (((int64_t)C + 63) / 64)) throw Other();
    const float *const px = f32(x.data_ptr());
    uint64_t *const pc = u64(cols);
    void *const pws = ws.data_ptr();
    const size_t nws = (size_t)ws.numel();
    return launch([&](void *s) { return lib.im2col(px, N, C, H, W, kH, kW, st[0], st[1], pd[0], pd[1], pc, pws, nws, s); });
  });
}

// x, w, scale, bias, stride, pad, out
template <class Out>
PyObject *first_layer(Args &v, bnn_status (*call)(const float *, const float *, int, int, int, int, int, int, int, int, int, int,
                                                  int, const float *, const float *, Out *, void *)) {
  const at::Tensor &x = v.tensor(kFloat, 4), &w = v.tensor(kFloat, 4);
  const float *const sc = f32(v.pointer()), *const bi = f32(v.pointer());
  int st[2], pd[2];
  v.pair(st);
  v.pair(pd);
  Out *const out = static_cast<Out *>(v.tensor().data_ptr());
  const int N = size(x, 0), C = size(x, 1), H = size(x, 2), W = size(x, 3), D = size(w, 0), kH = size(w, 2), kW = size(w, 3);
  const float *const px = f32(x.data_ptr()), *const pw = f32(w.data_ptr());
  return launch([&](void *s) { return call(px, pw, N, C, H, W, D, kH, kW, st[0], st[1], pd[0], pd[1], sc, bi, out, s); });
}

PyObject *f32_sign(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, 7, [](Args &v) { return first_layer(v, lib.f32_sign); });
}

PyObject *conv2d_f32(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, 7, [](Args &v) { return first_layer(v, lib.f32); });
}

PyObject *maxpool(PyObject *, PyObject *const *a, Py_ssize_t n) {  // in, out_i32, out_f32, scale, bias
  return guarded(a, n, 5, [](Args &v) {
    const at::Tensor &t = v.tensor(kInt, 4);
    int32_t *const oi = i32(v.pointer());
    float *const of = f32(v.pointer());
    const float *const sc = f32(v.pointer()), *const bi = f32(v.pointer());
    if (!t.is_contiguous()) throw Other();
    const int N = size(t, 0), D = size(t, 1), H = size(t, 2), W = size(t, 3);
    const int32_t *const p = i32(t.data_ptr());
    return launch([&](void *s) { return lib.maxpool(p, N, D, H, W, oi, of, sc, bi, s); });
  });
}

PyObject *fc(PyObject *, PyObject *const *a, Py_ssize_t n) {  // x, w, bias, sign_input, out
  return guarded(a, n, 5, [](Args &v) {
    const at::Tensor &x = v.tensor(kFloat, 2), &w = v.tensor(kFloat, 2);
    const float *const bi = f32(v.pointer());
    const int sign = v.small();
    float *const out = f32(v.tensor().data_ptr());
    const int64_t M = x.size(0), K = x.size(1), N = w.size(0);
    const float *const px = f32(x.data_ptr()), *const pw = f32(w.data_ptr());
    return launch([&](void *s) { return lib.fc(px, pw, bi, M, K, N, sign, out, s); });
  });
}

PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  constexpr Py_ssize_t want = sizeof(Library) / sizeof(void *);
  static_assert(want == sizeof(names) / sizeof(names[0]), "an address for every name");
  void *p[want];
  if (n != want) {
    PyErr_SetString(PyExc_TypeError, "one address per name");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < want; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an address");
      return nullptr;
    }
  }
  memcpy(&lib, p, sizeof lib);
  Py_RETURN_NONE;
}

#define BNN_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {BNN_METHOD(bind), BNN_METHOD(gemm), BNN_METHOD(epilogue), BNN_METHOD(encode), BNN_METHOD(conv2d),
                         BNN_METHOD(conv2d_packed), BNN_METHOD(im2col), BNN_METHOD(f32_sign), BNN_METHOD(conv2d_f32),
                         BNN_METHOD(maxpool), BNN_METHOD(fc), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tensorcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tensorcall() {
  PyObject *m = PyModule_Create(&module);
  if (!m) return nullptr;
  PyObject *t = PyTuple_New(sizeof(names) / sizeof(names[0]));
  if (!t) return nullptr;
  for (size_t i = 0; i < sizeof(names) / sizeof(names[0]); ++i) PyTuple_SET_ITEM(t, i, PyUnicode_FromString(names[i]));
  if (PyModule_AddObject(m, "names", t) < 0) return nullptr;
  if (PyModule_AddStringConstant(m, "built_for", BNN_BUILT_FOR) < 0) return nullptr;
  return m;
}
