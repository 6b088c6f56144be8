// The binding's calls, native: the checks of binding.py on well-formed arguments, the pointers and strides taken from
// the tensors, and the C entry point called with the GIL released.
//
// In Python a product's checks, its twelve ctypes arguments and the stream took 3.5 us beside the 3.5 us of the launch itself, and
// the small passes are bound by what issues their launches (a two-layer step, 256 x 1024-1024-10: 60 us of host time for 40 us
// of kernels).  Here they take about half a microsecond: the step's launches, nine then, were issued in 28 us, and it took 41.5 us
// instead of 58.7 (eight launches now, 39.5 us).
//
// A function returns the status of its entry point, or None where anything is not plainly as it should be: another type or
// shape, a tensor subclass, an active torch function mode, a host tensor, the library not loaded yet.  The caller then goes
// through the Python checks, which know every accepted form and word every error.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <string.h>
#include <vector>
#include "mpt.h"

namespace {

struct Refused {};                                                    // the Python checks are to have a look

// ---------------------------------------------------------------- entry points, by the addresses that the loaded library gives
#define MPT_CALLS(X)                                                                                                             \
  X(mpt_gemm_fwd) X(mpt_gemm_fwd_relu) X(mpt_gemm_dgrad) X(mpt_gemm_dgrad_relu) X(mpt_gemm_wgrad) X(mpt_conv3x3_fwd)               \
  X(mpt_conv3x3_dgrad) X(mpt_conv3x3_wgrad) X(mpt_unscale_check) X(mpt_master_update) X(mpt_master_update_multi)                  \
  X(mpt_loss_scale_update_dev) X(mpt_softmax_xent_scaled) X(mpt_add_fp16) X(mpt_relu_bwd) X(mpt_bn_stats) X(mpt_bn_apply)         \
  X(mpt_bn_bwd_reduce) X(mpt_bn_bwd_apply) X(mpt_lstm_cell_fwd) X(mpt_lstm_cell_bwd) X(mpt_master_update_fused)                    \
  X(mpt_optimizer_update) X(mpt_grad_sumsq) X(mpt_clip_factor) X(mpt_grad_stats) X(mpt_relu_fwd)
#define X(name) decltype(&::name) p_##name = nullptr;
MPT_CALLS(X)
#undef X
PyObject* params_type = nullptr;                                      // binding.mpt_opt_params

// ---------------------------------------------------------------- arguments
// A tensor as the checks below see it.  Sizes and strides are read once; what throws (symbolic sizes, no storage) ends in Refused.
struct T {
  const at::Tensor* t = nullptr;
  explicit operator bool() const { return t != nullptr; }
  int64_t dim() const { return t->dim(); }
  int64_t size(int k) const { return t->sizes()[k]; }
  int64_t numel() const { return t->numel(); }
  at::ScalarType type() const { return t->scalar_type(); }
  template <class P> P* ptr() const { return t == nullptr ? nullptr : static_cast<P*>(t->data_ptr()); }
  uint16_t* h() const { return ptr<uint16_t>(); }
  float* f() const { return ptr<float>(); }
  int64_t ld() const { return t == nullptr ? 0 : t->strides()[0]; }
};

void want(bool ok) { if (!ok) throw Refused{}; }

T optional(PyObject* o) {
  if (o == Py_None) return T{};
  want(THPVariable_CheckExact(o));
  const at::Tensor& t = THPVariable_Unpack(o);
  want(t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && !t.unsafeGetTensorImpl()->is_python_dispatch());
  return T{&t};
}
T tensor(PyObject* o) {
  want(o != Py_None);
  return optional(o);
}
// row-major rows of the shape, as binding._mat takes them at once
T mat(PyObject* o, int64_t rows, int64_t cols, at::ScalarType type = at::kHalf) {
  const T t = tensor(o);
  want(t.type() == type && t.dim() == 2 && t.size(0) == rows && t.size(1) == cols && t.t->strides()[1] == 1 && t.ld() >= cols);
  return t;
}
T any_mat(PyObject* o) {                                              // FP16, its shape is the call's
  const T t = tensor(o);
  want(t.dim() == 2);
  return mat(o, t.size(0), t.size(1));
}
T flat(PyObject* o, at::ScalarType type, int64_t numel, bool required = true) {
  const T t = optional(o);
  want(t || !required);
  if (t) want(t.type() == type && t.numel() == numel && t.t->is_contiguous());
  return t;
}
T one(PyObject* o, at::ScalarType type, int64_t numel = 1) {          // optional, of so many elements, any strides
  const T t = optional(o);
  if (t) want(t.type() == type && t.numel() == numel);
  return t;
}
struct Ws { void* p; size_t bytes; };
Ws workspace(PyObject* o) {
  const T t = optional(o);
  if (!t) return {nullptr, 0};
  want(t.t->is_contiguous());
  return {t.t->data_ptr(), (size_t)t.numel() * t.t->element_size()};
}
// FP16 or FP32, dense: whether it is FP32
T gradient(PyObject* o, int* fp32) {
  const T t = tensor(o);
  want((t.type() == at::kHalf || t.type() == at::kFloat) && t.t->is_contiguous());
  *fp32 = t.type() == at::kFloat;
  return t;
}
float number(PyObject* o) {                                          // what has a value as a float, as ctypes takes it: numpy's classes too
  const double d = PyFloat_AsDouble(o);
  want(!(d == -1.0 && PyErr_Occurred()));
  return (float)d;
}
int truth(PyObject* o) {
  const int t = PyObject_IsTrue(o);
  want(t >= 0);
  return t;
}

// ---------------------------------------------------------------- the call
typedef PyObject* const* Args;
template <class F, class... A>
int call(F f, A... a) {                                               // on the current device's current stream, the GIL released as by ctypes
  want(f != nullptr);
  void* const s = c10::hip::getCurrentHIPStream().stream();
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = f(s, a...);
  Py_END_ALLOW_THREADS
  return st;
}

template <int N, int (*BODY)(Args)>
PyObject* guarded(PyObject*, Args a, Py_ssize_t n) {
  try {
    if (n == N && !at::impl::torch_function_mode_enabled()) return PyLong_FromLong(BODY(a));
  } catch (const Refused&) {
  } catch (...) {                                                     // the Python path meets it again and reports it
  }
  PyErr_Clear();
  Py_RETURN_NONE;
}

template <decltype(&p_mpt_gemm_fwd) P>
int gemm_fwd(Args a) {                                                // X, W, Y, ws
  const T X = any_mat(a[0]), W = tensor(a[1]);
  want(W.dim() == 2);
  const int64_t M = X.size(0), K = X.size(1), N = W.size(1);
  mat(a[1], K, N);
  const T Y = mat(a[2], M, N);
  const Ws ws = workspace(a[3]);
  return call(*P, M, N, K, X.h(), X.ld(), W.h(), W.ld(), Y.h(), Y.ld(), ws.p, ws.bytes);
}
int gemm_dgrad(Args a) {                                              // dY, W, dX, ws
  const T dY = any_mat(a[0]), W = tensor(a[1]);
  want(W.dim() == 2);
  const int64_t M = dY.size(0), N = dY.size(1), K = W.size(0);
  mat(a[1], K, N);
  const T dX = mat(a[2], M, K);
  const Ws ws = workspace(a[3]);
  return call(p_mpt_gemm_dgrad, M, N, K, dY.h(), dY.ld(), W.h(), W.ld(), dX.h(), dX.ld(), ws.p, ws.bytes);
}
int gemm_dgrad_relu(Args a) {                                         // dY, W, H, dX, ws
  const T dY = any_mat(a[0]), W = tensor(a[1]);
  want(W.dim() == 2);
  const int64_t M = dY.size(0), N = dY.size(1), K = W.size(0);
  mat(a[1], K, N);
  const T H = mat(a[2], M, K), dX = mat(a[3], M, K);
  const Ws ws = workspace(a[4]);
  return call(p_mpt_gemm_dgrad_relu, M, N, K, dY.h(), dY.ld(), W.h(), W.ld(), H.h(), H.ld(), dX.h(), dX.ld(), ws.p, ws.bytes);
}
int gemm_wgrad(Args a) {                                              // X, dY, dW, accumulate, flag, ws
  const T X = any_mat(a[0]), dY = tensor(a[1]), dW = tensor(a[2]);
  want(dY.dim() == 2);
  const int64_t M = X.size(0), K = X.size(1), N = dY.size(1);
  mat(a[1], M, N);
  const int fp32 = dW.type() == at::kFloat, accumulate = truth(a[3]);
  mat(a[2], K, N, fp32 ? at::kFloat : at::kHalf);
  want(fp32 || !accumulate);
  const T flag = one(a[4], at::kInt);
  const Ws ws = workspace(a[5]);
  return call(p_mpt_gemm_wgrad, M, N, K, X.h(), X.ld(), dY.h(), dY.ld(), dW.ptr<void>(), dW.ld(), fp32, accumulate, flag.ptr<uint32_t>(), ws.p, ws.bytes);
}

struct Conv { int64_t Nb, H, W, C, Kf; };
Conv conv_shapes(PyObject* xo, PyObject* wo, PyObject* yo) {
  const T x = tensor(xo), w = tensor(wo), y = tensor(yo);
  want(x.dim() == 4 && w.dim() == 4 && y.dim() == 4);
  const Conv c{x.size(0), x.size(1), x.size(2), x.size(3), w.size(0)};
  want(w.size(1) == 3 && w.size(2) == 3 && w.size(3) == c.C && y.size(0) == c.Nb && y.size(1) == c.H && y.size(2) == c.W && y.size(3) == c.Kf);
  for (const T& t : {x, w, y}) want(t.type() == at::kHalf && t.t->is_contiguous());
  return c;
}
int conv_fwd(Args a) {                                                // x, w, y, ws
  const Conv c = conv_shapes(a[0], a[1], a[2]);
  const Ws ws = workspace(a[3]);
  return call(p_mpt_conv3x3_fwd, c.Nb, c.H, c.W, c.C, c.Kf, tensor(a[0]).h(), tensor(a[1]).h(), tensor(a[2]).h(), ws.p, ws.bytes);
}
int conv_dgrad(Args a) {                                              // dy, w, dx, ws
  const Conv c = conv_shapes(a[2], a[1], a[0]);
  const Ws ws = workspace(a[3]);
  return call(p_mpt_conv3x3_dgrad, c.Nb, c.H, c.W, c.C, c.Kf, tensor(a[0]).h(), tensor(a[1]).h(), tensor(a[2]).h(), ws.p, ws.bytes);
}
int conv_wgrad(Args a) {                                              // x, dy, dw, flag, ws
  const Conv c = conv_shapes(a[0], a[2], a[1]);
  const T flag = one(a[3], at::kInt);
  const Ws ws = workspace(a[4]);
  return call(p_mpt_conv3x3_wgrad, c.Nb, c.H, c.W, c.C, c.Kf, tensor(a[0]).h(), tensor(a[1]).h(), tensor(a[2]).h(), flag.ptr<uint32_t>(), ws.p, ws.bytes);
}

int unscale_check(Args a) {                                           // grad, inv_scale, flag, g32_out
  int fp32;
  const T g = gradient(a[0], &fp32), flag = one(a[2], at::kInt), out = flat(a[3], at::kFloat, g.numel(), false);
  want((bool)flag);
  return call(p_mpt_unscale_check, g.ptr<const void>(), fp32, (size_t)g.numel(), number(a[1]), out.f(), flag.ptr<uint32_t>());
}
// w32, momentum, gradient and FP16 copy of one parameter tensor
mpt_update_item update_item(PyObject* w, PyObject* m, PyObject* g, PyObject* h, int* fp32) {
  const T w32 = tensor(w), grad = gradient(g, fp32);
  const int64_t n = w32.numel();
  want(w32.type() == at::kFloat && w32.t->is_contiguous() && grad.numel() == n);
  return mpt_update_item{w32.f(), flat(m, at::kFloat, n, false).f(), grad.ptr<const void>(), flat(h, at::kHalf, n).h(), (size_t)n};
}
T scaler(PyObject* o) { return one(o, at::kByte, sizeof(mpt_scaler)); }
int master_update(Args a) {                                           // w32, m32, grad, w16, inv_scale, lr, momentum, flag, scaler_dev
  int fp32;
  const mpt_update_item u = update_item(a[0], a[1], a[2], a[3], &fp32);
  const T flag = one(a[7], at::kInt), sc = scaler(a[8]);
  return call(p_mpt_master_update, u.n, u.w32_dev, u.m32_dev, u.grad_dev, fp32, u.w16_dev, number(a[4]), sc.ptr<mpt_scaler>(), number(a[5]), number(a[6]),
              flag.ptr<uint32_t>());
}
int master_update_multi(Args a) {                                     // tensors, inv_scale, lr, momentum, flag, scaler_dev
  want(PyList_CheckExact(a[0]) || PyTuple_CheckExact(a[0]));
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(a[0]);
  want(n > 0 && n <= 0x7FFFFFFF);
  std::vector<mpt_update_item> items;
  items.reserve(n);
  int first = 0;
  for (Py_ssize_t k = 0; k < n; ++k) {
    PyObject* e = PySequence_Fast_GET_ITEM(a[0], k);
    want((PyList_CheckExact(e) || PyTuple_CheckExact(e)) && PySequence_Fast_GET_SIZE(e) == 4);
    PyObject** f = PySequence_Fast_ITEMS(e);
    int fp32;
    items.push_back(update_item(f[0], f[1], f[2], f[3], &fp32));
    if (k == 0) first = fp32;
    want(fp32 == first && (items[k].m32_dev == nullptr) == (items[0].m32_dev == nullptr) && (f[1] == Py_None) == (items[0].m32_dev == nullptr));
  }
  const T flag = one(a[4], at::kInt), sc = scaler(a[5]);
  return call(p_mpt_master_update_multi, (int)n, (const mpt_update_item*)items.data(), first, number(a[1]), sc.ptr<mpt_scaler>(), number(a[2]), number(a[3]),
              flag.ptr<uint32_t>());
}
int master_update_fused(Args a) {                                     // w32_in, m32_in, grad, w32_out, m32_out, w16_out, inv_scale, lr, momentum, flag, scaler_dev
  int fp32;
  const mpt_update_item in = update_item(a[0], a[1], a[2], a[5], &fp32);
  const int64_t n = (int64_t)in.n;
  const T out = flat(a[3], at::kFloat, n), m = flat(a[4], at::kFloat, n, false), flag = one(a[9], at::kInt), sc = scaler(a[10]);
  want(flag && (a[1] == Py_None) == (a[4] == Py_None));
  return call(p_mpt_master_update_fused, in.n, in.w32_dev, in.m32_dev, in.grad_dev, fp32, out.f(), m.f(), in.w16_dev, number(a[6]), sc.ptr<mpt_scaler>(),
              number(a[7]), number(a[8]), flag.ptr<uint32_t>());
}
int optimizer_update(Args a) {                                        // kind, hp, w32, state1, state2, grad, w16, inv_scale, flag, scaler_dev
  static const char* const kinds[] = {"momentum", "nesterov", "adagrad", "adam"};
  want(PyUnicode_CheckExact(a[0]));
  int kind = 0;
  while (kind < 4 && PyUnicode_CompareWithASCIIString(a[0], kinds[kind]) != 0) ++kind;
  want(kind < 4 && (PyObject*)Py_TYPE(a[1]) == params_type && a[3] != Py_None && (kind != 3 || a[4] != Py_None));
  mpt_opt_params hp;
  Py_buffer view;
  want(PyObject_GetBuffer(a[1], &view, PyBUF_SIMPLE) == 0);
  const bool whole = view.len == (Py_ssize_t)sizeof(hp);
  if (whole) memcpy(&hp, view.buf, sizeof(hp));
  PyBuffer_Release(&view);
  want(whole);
  int fp32;
  const mpt_update_item u = update_item(a[2], a[3], a[5], a[6], &fp32);
  const T second = flat(a[4], at::kFloat, (int64_t)u.n, false), flag = one(a[8], at::kInt), sc = scaler(a[9]);
  return call(p_mpt_optimizer_update, u.n, kind, (const mpt_opt_params*)&hp, u.w32_dev, u.m32_dev, second.f(), u.grad_dev, fp32, u.w16_dev, number(a[7]),
              sc.ptr<mpt_scaler>(), flag.ptr<uint32_t>());
}
int grad_sumsq(Args a) {                                              // grad, inv_scale, sumsq, ws, flag, accumulate, scaler_dev
  int fp32;
  const T g = gradient(a[0], &fp32), sum = one(a[2], at::kDouble), flag = one(a[4], at::kInt), sc = scaler(a[6]);
  want((bool)sum);
  const Ws ws = workspace(a[3]);
  return call(p_mpt_grad_sumsq, g.ptr<const void>(), fp32, (size_t)g.numel(), number(a[1]), sc.ptr<mpt_scaler>(), truth(a[5]), sum.ptr<double>(),
              flag.ptr<uint32_t>(), ws.p, ws.bytes);
}
int clip_factor(Args a) {                                             // sumsq, max_norm, factor, norm
  const T sum = one(a[0], at::kDouble), factor = one(a[2], at::kFloat), norm = one(a[3], at::kFloat);
  want(sum && factor);
  return call(p_mpt_clip_factor, sum.ptr<double>(), number(a[1]), factor.f(), norm.f());
}
int grad_stats(Args a) {                                              // grad, hist, absmax_bits, accumulate
  const T g = tensor(a[0]), most = one(a[2], at::kInt);
  flat(a[0], at::kHalf, g.numel());
  want((bool)most);
  return call(p_mpt_grad_stats, g.h(), (size_t)g.numel(), truth(a[3]), flat(a[1], at::kLong, 42).ptr<uint64_t>(), most.ptr<uint32_t>());
}
int loss_scale_update_dev(Args a) {                                   // scaler_dev, flag
  const T sc = scaler(a[0]), flag = one(a[1], at::kInt);
  want(sc && flag);
  return call(p_mpt_loss_scale_update_dev, sc.ptr<mpt_scaler>(), flag.ptr<uint32_t>());
}

int softmax(Args a) {                                                 // logits, labels, scale, dlogits, loss, row_loss
  const T z = any_mat(a[0]);
  const int64_t B = z.size(0), C = z.size(1);
  const T lab = flat(a[1], at::kInt, B), d = mat(a[3], B, C), loss = one(a[4], at::kFloat), rows = flat(a[5], at::kFloat, B, false);
  want(!loss || rows);
  return call(p_mpt_softmax_xent_scaled, B, C, z.h(), z.ld(), lab.ptr<int32_t>(), number(a[2]), loss.f(), rows.f(), d.h(), d.ld());
}
int add_fp16(Args a) {                                                // a, b, out
  const T x = tensor(a[0]);
  const int64_t n = x.numel();
  flat(a[0], at::kHalf, n);
  return call(p_mpt_add_fp16, (size_t)n, x.h(), flat(a[1], at::kHalf, n).h(), flat(a[2], at::kHalf, n).h());
}
int relu_fwd(Args a) {                                                // y, h
  const T y = tensor(a[0]);
  const int64_t n = y.numel();
  flat(a[0], at::kHalf, n);
  return call(p_mpt_relu_fwd, (size_t)n, y.h(), flat(a[1], at::kHalf, n).h());
}
int relu_bwd(Args a) {                                                // dh, y, dy
  const T y = tensor(a[1]);
  const int64_t n = y.numel();
  flat(a[1], at::kHalf, n);
  return call(p_mpt_relu_bwd, (size_t)n, flat(a[0], at::kHalf, n).h(), y.h(), flat(a[2], at::kHalf, n).h());
}

int bn_stats(Args a) {                                                // x, mean, var, ws
  const T x = any_mat(a[0]);
  const int64_t P = x.size(0), C = x.size(1);
  const T mean = flat(a[1], at::kFloat, C), var = flat(a[2], at::kFloat, C);
  const Ws ws = workspace(a[3]);
  return call(p_mpt_bn_stats, P, C, x.h(), x.ld(), mean.f(), var.f(), ws.p, ws.bytes);
}
int bn_apply(Args a) {                                                // x, mean, var, gamma, beta, eps, y, relu
  const T x = any_mat(a[0]);
  const int64_t P = x.size(0), C = x.size(1);
  const T y = mat(a[6], P, C);
  return call(p_mpt_bn_apply, P, C, x.h(), x.ld(), flat(a[1], at::kFloat, C).f(), flat(a[2], at::kFloat, C).f(), flat(a[3], at::kFloat, C).f(),
              flat(a[4], at::kFloat, C).f(), number(a[5]), truth(a[7]), y.h(), y.ld());
}
int bn_bwd_reduce(Args a) {                                           // x, dy, mean, var, eps, dgamma, dbeta, ws
  const T x = any_mat(a[0]);
  const int64_t P = x.size(0), C = x.size(1);
  const T dy = mat(a[1], P, C);
  const Ws ws = workspace(a[7]);
  return call(p_mpt_bn_bwd_reduce, P, C, x.h(), x.ld(), dy.h(), dy.ld(), flat(a[2], at::kFloat, C).f(), flat(a[3], at::kFloat, C).f(), number(a[4]),
              flat(a[5], at::kFloat, C).f(), flat(a[6], at::kFloat, C).f(), ws.p, ws.bytes);
}
int bn_bwd_apply(Args a) {                                            // x, dy, mean, var, gamma, eps, dgamma, dbeta, dx
  const T x = any_mat(a[0]);
  const int64_t P = x.size(0), C = x.size(1);
  const T dy = mat(a[1], P, C), dx = mat(a[8], P, C);
  return call(p_mpt_bn_bwd_apply, P, C, x.h(), x.ld(), dy.h(), dy.ld(), flat(a[2], at::kFloat, C).f(), flat(a[3], at::kFloat, C).f(),
              flat(a[4], at::kFloat, C).f(), number(a[5]), flat(a[6], at::kFloat, C).f(), flat(a[7], at::kFloat, C).f(), dx.h(), dx.ld());
}

T optional_mat(PyObject* o, int64_t rows, int64_t cols) { return o == Py_None ? T{} : mat(o, rows, cols); }
int lstm_cell_fwd(Args a) {                                           // gx, gr, bias, c_prev, act, c, h
  const T cp = any_mat(a[3]);
  const int64_t B = cp.size(0), H = cp.size(1);
  const T gx = mat(a[0], B, 4 * H), gr = optional_mat(a[1], B, 4 * H), bias = flat(a[2], at::kFloat, 4 * H, false), act = mat(a[4], B, 4 * H),
          c = mat(a[5], B, H), h = mat(a[6], B, H);
  return call(p_mpt_lstm_cell_fwd, B, H, gx.h(), gx.ld(), gr.h(), gr.ld(), bias.f(), cp.h(), cp.ld(), act.h(), act.ld(), c.h(), c.ld(), h.h(), h.ld());
}
int lstm_cell_bwd(Args a) {                                           // dh, dc_next, act, c, c_prev, da, dc_prev
  const T c = any_mat(a[3]);
  const int64_t B = c.size(0), H = c.size(1);
  const T dh = mat(a[0], B, H), dn = optional_mat(a[1], B, H), act = mat(a[2], B, 4 * H), cp = mat(a[4], B, H), da = mat(a[5], B, 4 * H), dp = mat(a[6], B, H);
  return call(p_mpt_lstm_cell_bwd, B, H, dh.h(), dh.ld(), dn.h(), dn.ld(), act.h(), act.ld(), c.h(), c.ld(), cp.h(), cp.ld(), da.h(), da.ld(), dp.h(), dp.ld());
}

// The entry points' addresses, by name, from the library that the binding loaded; and its class of the optimizers' parameters.
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *addresses, *params;
  if (!PyArg_ParseTuple(args, "O!O!", &PyDict_Type, &addresses, &PyType_Type, &params)) return nullptr;
  Py_INCREF(params);
  Py_XDECREF(params_type);
  params_type = params;
#define X(name)                                                                                          \
  {                                                                                                      \
    PyObject* o = PyDict_GetItemString(addresses, #name);                                                \
    void* p = o == nullptr ? nullptr : PyLong_AsVoidPtr(o);                                              \
    if (p == nullptr) {                                                                                  \
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);                                     \
      return nullptr;                                                                                    \
    }                                                                                                    \
    p_##name = reinterpret_cast<decltype(&::name)>(p);                                                   \
  }
  MPT_CALLS(X)
#undef X
  Py_RETURN_NONE;
}

#define M(name, n, ...) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(static_cast<PyObject* (*)(PyObject*, Args, Py_ssize_t)>(guarded<n, __VA_ARGS__>))), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    M("gemm_fwd", 4, gemm_fwd<&p_mpt_gemm_fwd>), M("gemm_fwd_relu", 4, gemm_fwd<&p_mpt_gemm_fwd_relu>), M("gemm_dgrad", 4, gemm_dgrad),
    M("gemm_dgrad_relu", 5, gemm_dgrad_relu), M("gemm_wgrad", 6, gemm_wgrad), M("conv3x3_fwd", 4, conv_fwd), M("conv3x3_dgrad", 4, conv_dgrad),
    M("conv3x3_wgrad", 5, conv_wgrad), M("unscale_check", 4, unscale_check), M("master_update", 9, master_update),
    M("master_update_multi", 6, master_update_multi), M("loss_scale_update_dev", 2, loss_scale_update_dev), M("softmax_xent_scaled", 6, softmax),
    M("add_fp16", 3, add_fp16), M("relu_bwd", 3, relu_bwd), M("bn_stats", 4, bn_stats), M("bn_apply", 8, bn_apply), M("bn_bwd_reduce", 8, bn_bwd_reduce),
    M("bn_bwd_apply", 9, bn_bwd_apply), M("lstm_cell_fwd", 7, lstm_cell_fwd), M("lstm_cell_bwd", 7, lstm_cell_bwd),
    M("master_update_fused", 11, master_update_fused), M("optimizer_update", 10, optimizer_update), M("grad_sumsq", 7, grad_sumsq), M("clip_factor", 4, clip_factor),
    M("grad_stats", 4, grad_stats), M("relu_fwd", 2, relu_fwd), {nullptr, nullptr, 0, nullptr}};
#undef M
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// `torch`: the torch whose headers this was compiled against, from the build.  The tensors' fields are read by inlined code, at places that
// another torch may have elsewhere: the binding compares before it calls anything here.
PyMODINIT_FUNC PyInit__calls(void) {
  PyObject* m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "torch", MPT_TORCH) != 0) Py_CLEAR(m);
  return m;
}
