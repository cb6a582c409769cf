// Native half of the Python binding: takes torch tensors, checks them, allocates outputs, and calls the entry
// point of the same name in the C ABI library on the current stream.  Argument marshalling only.
//
// A call of the library enqueues one to five kernels, which the runtime takes 2.3 us each to accept; marshalled in
// Python (tensor checks, ctypes conversion, torch.empty, torch.cuda.current_stream) a call cost 4 to 7 us more than
// that, half of the time of the smallest ones.
#include <Python.h>
#include <dlfcn.h>

#include <string>

#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/amq.h"

namespace {

// ---- the library's entry points, resolved in the library file the binding names
#define AMQ_ENTRIES(X)                                                                                              \
  X(amq_wpr) X(amq_status_string) X(amq_last_hip_error) X(amq_quantize_weights) X(amq_quantize_weights_ex)          \
  X(amq_quantize_activations) X(amq_binary_gemm) X(amq_binary_gemv) X(amq_lstm_workspace_bytes) X(amq_lstm_step)    \
  X(amq_lstm_step_static) X(amq_lstm_step_packed) X(amq_lstm_sequence_workspace_bytes) X(amq_lstm_sequence)         \
  X(amq_gru_workspace_bytes) X(amq_gru_step) X(amq_gru_sequence_workspace_bytes) X(amq_gru_sequence)                \
  X(amq_embedding_lookup) X(amq_log_softmax) X(amq_softmax_layer_workspace_bytes) X(amq_softmax_layer)              \
  X(amq_lm_workspace_bytes) X(amq_lm_step) X(amq_lm_sequence_workspace_bytes) X(amq_lm_sequence)                    \
  X(amq_lm_sequence_score_workspace_bytes) X(amq_lm_sequence_score) X(amq_dequantize)      \
  X(amq_quantize_reconstruct)

struct Api {
#define AMQ_MEMBER(name) decltype(&::name) name = nullptr;
  AMQ_ENTRIES(AMQ_MEMBER)
#undef AMQ_MEMBER
} api;
PyObject* amq_error = nullptr;

// A Python exception is already set.
struct PythonError {};

[[noreturn]] void fail(PyObject* type, const std::string& msg) {
  PyErr_SetString(type, msg.c_str());
  throw PythonError();
}

const char* dtype_name(at::ScalarType t) {
  switch (t) {
    case at::kFloat: return "torch.float32";
    case at::kDouble: return "torch.float64";
    case at::kHalf: return "torch.float16";
    case at::kBFloat16: return "torch.bfloat16";
    case at::kInt: return "torch.int32";
    case at::kLong: return "torch.int64";
    case at::kByte: return "torch.uint8";
    default: return c10::toString(t);
  }
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) fail(amq_error, "expected a GPU tensor");
  return THPVariable_Unpack(o);
}

// The data pointer of a contiguous GPU tensor of the given type.
void* dev(const at::Tensor& t, at::ScalarType dt) {
  if (!t.is_cuda()) fail(amq_error, "expected a GPU tensor");
  if (t.scalar_type() != dt || !t.is_contiguous())
    fail(amq_error, std::string("expected a contiguous ") + dtype_name(dt) + " tensor, got " + dtype_name(t.scalar_type()));
  return t.data_ptr();
}
float* f32(PyObject* o) { return static_cast<float*>(dev(tensor(o), at::kFloat)); }
uint32_t* words(PyObject* o) { return static_cast<uint32_t*>(dev(tensor(o), at::kInt)); }
const int64_t* i64(PyObject* o) { return static_cast<const int64_t*>(dev(tensor(o), at::kLong)); }
float* f32_or_null(PyObject* o) { return o == Py_None ? nullptr : f32(o); }

int64_t integer(PyObject* o) {
  const int64_t v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw PythonError();
  return v;
}

const at::Tensor& shaped(PyObject* o, int64_t dims) {
  const at::Tensor& t = tensor(o);
  if (t.dim() != dims) fail(PyExc_ValueError, "expected a tensor of " + std::to_string(dims) + " dimensions, got " + std::to_string(t.dim()));
  return t;
}

at::Tensor make(at::IntArrayRef shape, at::ScalarType dt, const at::Tensor& like) {
  if (!like.is_cuda()) fail(amq_error, "expected a GPU tensor");
  return at::detail::empty_cuda(shape, dt, like.device(), std::nullopt);
}

PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }
PyObject* pair(PyObject* a, PyObject* b) {  // takes both references
  PyObject* r = (a && b) ? PyTuple_Pack(2, a, b) : nullptr;
  Py_XDECREF(a);
  Py_XDECREF(b);
  return r;
}
PyObject* again(PyObject* o) {
  Py_INCREF(o);
  return o;
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Calls f (an entry point, without the interpreter lock) and turns a status into an exception.
template <typename F>
void call(F f) {
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  if (st == AMQ_OK) return;
  std::string msg = api.amq_status_string(st);
  if (st == AMQ_ERR_HIP) msg += " (hipError " + std::to_string(api.amq_last_hip_error()) + ")";
  fail(amq_error, msg);
}

// A workspace: the caller's tensor, or a new one of `bytes`.
struct Workspace {
  at::Tensor own;
  void* ptr;
  size_t bytes;
  template <typename Q>
  Workspace(PyObject* o, const at::Tensor& like, Q query) {
    if (o == Py_None) {
      own = make({(int64_t)query()}, at::kByte, like);
      ptr = own.data_ptr();
      bytes = (size_t)own.numel();
    } else {
      const at::Tensor& t = tensor(o);
      ptr = t.data_ptr();
      bytes = (size_t)t.numel();
    }
  }
};

// An output: the caller's tensor, or a new one.
struct Output {
  PyObject* obj;  // owned
  Output(PyObject* o, at::IntArrayRef shape, const at::Tensor& like)
      : obj(o == Py_None ? wrap(make(shape, at::kFloat, like)) : again(o)) {
    if (!obj) throw PythonError();
  }
  ~Output() { Py_XDECREF(obj); }
  float* ptr() const { return f32(obj); }
  PyObject* take() {
    PyObject* o = obj;
    obj = nullptr;
    return o;
  }
};

// ---- entry points; arguments are positional, in the order of the Python functions that forward here

std::pair<at::Tensor, at::Tensor> quantize_matrix(const at::Tensor& W, int k, int T, int flags) {
  if (W.dim() != 2 || W.stride(1) != 1 || W.scalar_type() != at::kFloat || !W.is_cuda())
    fail(amq_error, "expected a 2-D float32 GPU tensor with unit column stride");
  const int64_t rows = W.size(0), cols = W.size(1), ld = W.stride(0);
  at::Tensor planes = make({k, rows, api.amq_wpr(cols)}, at::kInt, W);
  at::Tensor alpha = make({rows, k}, at::kFloat, W);
  const float* w = static_cast<const float*>(W.data_ptr());
  uint32_t* p = static_cast<uint32_t*>(planes.data_ptr());
  float* a = static_cast<float*>(alpha.data_ptr());
  void* s = stream();
  call([&] {
    return flags ? api.amq_quantize_weights_ex(w, rows, cols, ld, k, T, flags, p, a, s)
                 : api.amq_quantize_weights(w, rows, cols, ld, k, T, p, a, s);
  });
  return {std::move(planes), std::move(alpha)};
}

PyObject* quantize_weights(PyObject* const* a) {  // W, k, T, flags
  auto r = quantize_matrix(tensor(a[0]), (int)integer(a[1]), (int)integer(a[2]), (int)integer(a[3]));
  return pair(wrap(r.first), wrap(r.second));
}

PyObject* quantize_activations(PyObject* const* a) {  // X, k, T
  const at::Tensor& X = shaped(a[0], 2);
  const int64_t batch = X.size(0), n = X.size(1);
  const int k = (int)integer(a[1]), T = (int)integer(a[2]);
  const float* x = f32(a[0]);
  at::Tensor planes = make({k, batch, api.amq_wpr(n)}, at::kInt, X);
  at::Tensor beta = make({batch, k}, at::kFloat, X);
  uint32_t* p = static_cast<uint32_t*>(planes.data_ptr());
  float* b = static_cast<float*>(beta.data_ptr());
  void* s = stream();
  call([&] { return api.amq_quantize_activations(x, batch, n, k, T, p, b, s); });
  return pair(wrap(planes), wrap(beta));
}

PyObject* binary_gemm(PyObject* const* a) {  // Wp, alpha, n, Xp, beta, bias, Y
  const at::Tensor &W = shaped(a[0], 3), &X = shaped(a[3], 3);
  const int64_t m = W.size(1), n = integer(a[2]), batch = X.size(1);
  const int k_w = (int)W.size(0), k_a = (int)X.size(0), acc = a[6] != Py_None;
  const uint32_t *wp = words(a[0]), *xp = words(a[3]);
  const float *al = f32(a[1]), *be = f32(a[4]), *bi = f32_or_null(a[5]);
  Output Y(a[6], {batch, m}, W);
  float* y = Y.ptr();
  void* s = stream();
  call([&] { return api.amq_binary_gemm(wp, al, m, n, k_w, xp, be, batch, k_a, bi, acc, y, s); });
  return Y.take();
}

PyObject* binary_gemv(PyObject* const* a) {  // Wp, alpha, n, Xp, beta, bias, Y
  const at::Tensor &W = shaped(a[0], 3), &X = tensor(a[3]);
  const int64_t m = W.size(1), n = integer(a[2]);
  const int k_w = (int)W.size(0), k_a = (int)X.size(0), acc = a[6] != Py_None;
  const uint32_t *wp = words(a[0]), *xp = words(a[3]);
  const float *al = f32(a[1]), *be = f32(a[4]), *bi = f32_or_null(a[5]);
  Output Y(a[6], {1, m}, W);
  float* y = Y.ptr();
  void* s = stream();
  call([&] { return api.amq_binary_gemv(wp, al, m, n, k_w, xp, be, k_a, bi, acc, y, s); });
  return Y.take();
}

// Wxp, alpha_x, Whp, alpha_h, I, H: the head of every cell call
struct Cell {
  const uint32_t *wx, *wh;
  const float *ax, *ah;
  int64_t I, H;
  int k_w;
  explicit Cell(PyObject* const* a)
      : wx(words(a[0])), wh(words(a[2])), ax(f32(a[1])), ah(f32(a[3])), I(integer(a[4])), H(integer(a[5])),
        k_w((int)tensor(a[0]).size(0)) {}
};

PyObject* lstm_step(PyObject* const* a) {  // Cell, bias, x, h_prev, c_prev, k_a, T, ws, h_out, c_out
  const Cell w(a);
  const at::Tensor& x = tensor(a[7]);
  const int64_t B = x.size(0);
  const int k_a = (int)integer(a[10]), T = (int)integer(a[11]);
  const float *bi = f32_or_null(a[6]), *xp = f32(a[7]), *h = f32(a[8]), *c = f32(a[9]);
  Workspace ws(a[12], x, [&] { return api.amq_lstm_workspace_bytes(w.I, w.H, B, k_a); });
  Output ho(a[13], tensor(a[8]).sizes(), tensor(a[8])), co(a[14], tensor(a[9]).sizes(), tensor(a[9]));
  float *hp = ho.ptr(), *cp = co.ptr();
  void* s = stream();
  call([&] {
    return api.amq_lstm_step(w.wx, w.ax, w.wh, w.ah, w.I, w.H, w.k_w, bi, xp, h, c, B, k_a, T, hp, cp, ws.ptr, ws.bytes, s);
  });
  return pair(ho.take(), co.take());
}

PyObject* lstm_step_static(PyObject* const* a) {  // Cell, bias, x, h_prev, c_prev, k_a, T, h_out, c_out
  const Cell w(a);
  const int64_t B = tensor(a[7]).size(0);
  const int k_a = (int)integer(a[10]), T = (int)integer(a[11]);
  const float *bi = f32_or_null(a[6]), *xp = f32(a[7]), *h = f32(a[8]), *c = f32(a[9]);
  float *hp = f32(a[12]), *cp = f32(a[13]);
  void* s = stream();
  call([&] { return api.amq_lstm_step_static(w.wx, w.ax, w.wh, w.ah, w.I, w.H, w.k_w, bi, xp, h, c, B, k_a, T, hp, cp, s); });
  return pair(again(a[12]), again(a[13]));
}

PyObject* lstm_step_packed(PyObject* const* a) {  // Cell, bias, Xp, beta_x, Hp, beta_h, c_prev, h_out, c_out
  const Cell w(a);
  const at::Tensor& X = shaped(a[7], 3);
  const int64_t B = X.size(1);
  const int k_a = (int)X.size(0);
  const float *bi = f32_or_null(a[6]), *bx = f32(a[8]), *bh = f32(a[10]), *c = f32(a[11]);
  const uint32_t *xp = words(a[7]), *hq = words(a[9]);
  const at::Tensor& cpv = tensor(a[11]);
  Output ho(a[12], cpv.sizes(), cpv), co(a[13], cpv.sizes(), cpv);
  float *hp = ho.ptr(), *cp = co.ptr();
  void* s = stream();
  call([&] {
    return api.amq_lstm_step_packed(w.wx, w.ax, w.wh, w.ah, w.I, w.H, w.k_w, bi, xp, bx, hq, bh, c, B, k_a, hp, cp, s);
  });
  return pair(ho.take(), co.take());
}

PyObject* lstm_sequence(PyObject* const* a) {  // Cell, bias, xs, h, c, k_a, T, ws, hs
  const Cell w(a);
  const at::Tensor& xs = shaped(a[7], 3);
  const int64_t steps = xs.size(0), B = xs.size(1);
  const int k_a = (int)integer(a[10]), T = (int)integer(a[11]);
  const float *bi = f32_or_null(a[6]), *xp = f32(a[7]);
  float *h = f32(a[8]), *c = f32(a[9]), *hs = f32_or_null(a[13]);
  Workspace ws(a[12], xs, [&] { return api.amq_lstm_sequence_workspace_bytes(w.I, w.H, B, k_a); });
  void* s = stream();
  call([&] {
    return api.amq_lstm_sequence(w.wx, w.ax, w.wh, w.ah, w.I, w.H, w.k_w, bi, xp, steps, h, c, B, k_a, T, hs, ws.ptr,
                                 ws.bytes, s);
  });
  return pair(again(a[8]), again(a[9]));
}

PyObject* gru_step(PyObject* const* a) {  // Cell, bias_x, bias_h, x, h_prev, k_a, T, ws, h_out
  const Cell w(a);
  const at::Tensor& x = tensor(a[8]);
  const int64_t B = x.size(0);
  const int k_a = (int)integer(a[10]), T = (int)integer(a[11]);
  const float *bx = f32_or_null(a[6]), *bh = f32_or_null(a[7]), *xp = f32(a[8]), *h = f32(a[9]);
  Workspace ws(a[12], x, [&] { return api.amq_gru_workspace_bytes(w.I, w.H, B, k_a); });
  Output ho(a[13], tensor(a[9]).sizes(), tensor(a[9]));
  float* hp = ho.ptr();
  void* s = stream();
  call([&] {
    return api.amq_gru_step(w.wx, w.ax, w.wh, w.ah, w.I, w.H, w.k_w, bx, bh, xp, h, B, k_a, T, hp, ws.ptr, ws.bytes, s);
  });
  return ho.take();
}

PyObject* gru_sequence(PyObject* const* a) {  // Cell, bias_x, bias_h, xs, h, k_a, T, ws, hs
  const Cell w(a);
  const at::Tensor& xs = shaped(a[8], 3);
  const int64_t steps = xs.size(0), B = xs.size(1);
  const int k_a = (int)integer(a[10]), T = (int)integer(a[11]);
  const float *bx = f32_or_null(a[6]), *bh = f32_or_null(a[7]), *xp = f32(a[8]);
  float *h = f32(a[9]), *hs = f32_or_null(a[13]);
  Workspace ws(a[12], xs, [&] { return api.amq_gru_sequence_workspace_bytes(w.I, w.H, B, k_a); });
  void* s = stream();
  call([&] {
    return api.amq_gru_sequence(w.wx, w.ax, w.wh, w.ah, w.I, w.H, w.k_w, bx, bh, xp, steps, h, B, k_a, T, hs, ws.ptr,
                                ws.bytes, s);
  });
  return again(a[9]);
}

PyObject* embedding_lookup(PyObject* const* a) {  // Ep, alpha_e, n, ids
  const at::Tensor &E = shaped(a[0], 3), &ids = tensor(a[3]);
  const int64_t vocab = E.size(1), n = integer(a[2]), B = ids.size(0);
  const int k = (int)E.size(0);
  at::Tensor Xp = make({k, B, E.size(2)}, at::kInt, E);
  at::Tensor beta = make({B, k}, at::kFloat, E);
  const uint32_t* ep = words(a[0]);
  const float* ae = f32(a[1]);
  const int64_t* id = i64(a[3]);
  uint32_t* xp = static_cast<uint32_t*>(Xp.data_ptr());
  float* be = static_cast<float*>(beta.data_ptr());
  void* s = stream();
  call([&] { return api.amq_embedding_lookup(ep, ae, vocab, n, k, id, B, xp, be, s); });
  return pair(wrap(Xp), wrap(beta));
}

PyObject* log_softmax(PyObject* const* a) {  // Y, out
  const at::Tensor& Y = shaped(a[0], 2);
  const int64_t B = Y.size(0), V = Y.size(1);
  const float* y = f32(a[0]);
  Output out(a[1], Y.sizes(), Y);
  float* o = out.ptr();
  void* s = stream();
  call([&] { return api.amq_log_softmax(y, B, V, o, s); });
  return out.take();
}

PyObject* softmax_layer(PyObject* const* a) {  // Wsp, alpha_s, H, bias, h, k_a, T, ws, logprob
  const at::Tensor &W = shaped(a[0], 3), &ht = tensor(a[4]);
  const int64_t V = W.size(1), H = integer(a[2]), B = ht.size(0);
  const int k_w = (int)W.size(0), k_a = (int)integer(a[5]), T = (int)integer(a[6]);
  const uint32_t* wp = words(a[0]);
  const float *al = f32(a[1]), *bi = f32_or_null(a[3]), *h = f32(a[4]);
  Workspace ws(a[7], ht, [&] { return api.amq_softmax_layer_workspace_bytes(V, H, B, k_a); });
  Output lp(a[8], {B, V}, ht);
  float* o = lp.ptr();
  void* s = stream();
  call([&] { return api.amq_softmax_layer(wp, al, V, H, k_w, bi, h, B, k_a, T, o, ws.ptr, ws.bytes, s); });
  return lp.take();
}

// Ep, alpha_e, E, Wxp, alpha_x, Whp, alpha_h, H, bias, Wsp, alpha_s, bias_s, ids: the head of the language-model calls
struct Model {
  const uint32_t *ep, *wx, *wh, *wsp;
  const float *ae, *ax, *ah, *bias, *as, *bias_s;
  int64_t vocab, E, H, V;
  int k_w, k_ws;
  const int64_t* ids;
  explicit Model(PyObject* const* a) {
    vocab = tensor(a[0]).size(1);
    k_w = (int)tensor(a[3]).size(0);
    const at::Tensor& S = shaped(a[9], 3);
    k_ws = (int)S.size(0);
    V = S.size(1);
    ep = words(a[0]); ae = f32(a[1]); E = integer(a[2]);
    wx = words(a[3]); ax = f32(a[4]); wh = words(a[5]); ah = f32(a[6]); H = integer(a[7]); bias = f32_or_null(a[8]);
    wsp = words(a[9]); as = f32(a[10]); bias_s = f32_or_null(a[11]); ids = i64(a[12]);
  }
};

PyObject* lm_step(PyObject* const* a) {  // Model, h, c, k_a, k_as, T, ws, logprob
  const Model w(a);
  const at::Tensor& ht = tensor(a[13]);
  const int64_t B = tensor(a[12]).size(0);
  float *h = f32(a[13]), *c = f32(a[14]);
  const int k_a = (int)integer(a[15]), k_as = (int)integer(a[16]), T = (int)integer(a[17]);
  Workspace ws(a[18], ht, [&] { return api.amq_lm_workspace_bytes(w.E, w.H, w.V, B, k_a, k_as); });
  Output lp(a[19], {B, w.V}, ht);
  float* o = lp.ptr();
  void* s = stream();
  call([&] {
    return api.amq_lm_step(w.ep, w.ae, w.vocab, w.E, w.wx, w.ax, w.wh, w.ah, w.H, w.k_w, w.bias, w.wsp, w.as, w.V, w.k_ws,
                           w.bias_s, w.ids, h, c, B, k_a, k_as, T, o, ws.ptr, ws.bytes, s);
  });
  return lp.take();
}

PyObject* lm_sequence(PyObject* const* a) {  // Model, h, c, k_a, k_as, T, ws, logprob
  const Model w(a);
  const at::Tensor &ht = tensor(a[13]), &ids = shaped(a[12], 2);
  const int64_t steps = ids.size(0), B = ids.size(1);
  float *h = f32(a[13]), *c = f32(a[14]);
  const int k_a = (int)integer(a[15]), k_as = (int)integer(a[16]), T = (int)integer(a[17]);
  Workspace ws(a[18], ht, [&] { return api.amq_lm_sequence_workspace_bytes(w.E, w.H, w.V, B, k_a, k_as); });
  Output lp(a[19], {steps, B, w.V}, ht);
  float* o = lp.ptr();
  void* s = stream();
  call([&] {
    return api.amq_lm_sequence(w.ep, w.ae, w.vocab, w.E, w.wx, w.ax, w.wh, w.ah, w.H, w.k_w, w.bias, w.wsp, w.as, w.V,
                               w.k_ws, w.bias_s, w.ids, steps, h, c, B, k_a, k_as, T, o, ws.ptr, ws.bytes, s);
  });
  return lp.take();
}

PyObject* lm_sequence_score(PyObject* const* a) {  // Model, h, c, k_a, k_as, T, ws, out, targets
  const Model w(a);
  const at::Tensor &ht = tensor(a[13]), &ids = shaped(a[12], 2), &tg = tensor(a[20]);
  const int64_t steps = ids.size(0), B = ids.size(1);
  if (tg.sizes() != ids.sizes()) fail(amq_error, "targets must have the shape of ids");
  const int64_t* targets = i64(a[20]);
  float *h = f32(a[13]), *c = f32(a[14]);
  const int k_a = (int)integer(a[15]), k_as = (int)integer(a[16]), T = (int)integer(a[17]);
  Workspace ws(a[18], ht, [&] { return api.amq_lm_sequence_score_workspace_bytes(w.E, w.H, w.V, B, k_a, k_as); });
  Output out(a[19], {steps, B}, ht);
  float* o = out.ptr();
  void* s = stream();
  call([&] {
    return api.amq_lm_sequence_score(w.ep, w.ae, w.vocab, w.E, w.wx, w.ax, w.wh, w.ah, w.H, w.k_w, w.bias, w.wsp, w.as,
                                     w.V, w.k_ws, w.bias_s, w.ids, targets, steps, h, c, B, k_a, k_as, T, o, ws.ptr,
                                     ws.bytes, s);
  });
  return out.take();
}

at::Tensor dequantized(const at::Tensor& planes, const at::Tensor& alpha, int64_t cols, const at::Tensor& out) {
  if (out.dim() != 2 || out.stride(1) != 1 || out.scalar_type() != at::kFloat || !out.is_cuda())
    fail(amq_error, "expected a 2-D float32 GPU tensor with unit column stride");
  const int64_t rows = planes.size(1), ld = out.stride(0);
  const int k = (int)planes.size(0);
  const uint32_t* p = static_cast<const uint32_t*>(dev(planes, at::kInt));
  const float* al = static_cast<const float*>(dev(alpha, at::kFloat));
  float* o = static_cast<float*>(out.data_ptr());
  void* s = stream();
  call([&] { return api.amq_dequantize(p, al, rows, cols, k, o, ld, s); });
  return out;
}

PyObject* dequantize(PyObject* const* a) {  // planes, alpha, cols, out
  const at::Tensor& planes = shaped(a[0], 3);
  const int64_t cols = integer(a[2]);
  if (a[3] != Py_None) {
    dequantized(planes, tensor(a[1]), cols, tensor(a[3]));
    return again(a[3]);
  }
  return wrap(dequantized(planes, tensor(a[1]), cols, make({planes.size(1), cols}, at::kFloat, planes)));
}

// w -> w_hat with the straight-through gradient of Sec. 4: d f / d w = d f / d w_hat.
struct FakeQuantize : public torch::autograd::Function<FakeQuantize> {
  static at::Tensor forward(torch::autograd::AutogradContext*, const at::Tensor& W, int64_t k, int64_t T) {
    const at::Tensor w = W.detach().contiguous();
    if (w.dim() != 2 || w.scalar_type() != at::kFloat || !w.is_cuda())
      fail(amq_error, "expected a 2-D float32 GPU tensor with unit column stride");
    const int64_t rows = w.size(0), cols = w.size(1);
    at::Tensor out = make({rows, cols}, at::kFloat, w);
    const float* p = static_cast<const float*>(w.data_ptr());
    float* o = static_cast<float*>(out.data_ptr());
    void* s = stream();
    call([&] { return api.amq_quantize_reconstruct(p, rows, cols, cols, (int)k, (int)T, o, cols, s); });
    return out;
  }
  static torch::autograd::variable_list backward(torch::autograd::AutogradContext*,
                                                 const torch::autograd::variable_list& grad) {
    return {grad[0], at::Tensor(), at::Tensor()};
  }
};

PyObject* fake_quantize(PyObject* const* a) {  // W, k, T
  return wrap(FakeQuantize::apply(tensor(a[0]), integer(a[1]), integer(a[2])));
}

// ---- module

template <PyObject* (*F)(PyObject* const*), int N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  try {
    if (!api.amq_wpr) fail(PyExc_RuntimeError, "the library is not loaded");
    if (n != N) fail(PyExc_TypeError, "expected " + std::to_string(N) + " arguments, got " + std::to_string(n));
    return F(args);
  } catch (const PythonError&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

PyObject* load(PyObject*, PyObject* args) {  // path of the library, exception class
  const char* path;
  PyObject* err;
  if (!PyArg_ParseTuple(args, "sO", &path, &err)) return nullptr;
  void* lib = dlopen(path, RTLD_NOW | RTLD_LOCAL);
  if (!lib) {
    PyErr_SetString(PyExc_OSError, dlerror());
    return nullptr;
  }
  Api found;
  bool all = true;
#define AMQ_RESOLVE(name)                                                 \
  found.name = reinterpret_cast<decltype(found.name)>(dlsym(lib, #name)); \
  all = all && found.name;
  AMQ_ENTRIES(AMQ_RESOLVE)
#undef AMQ_RESOLVE
  if (!all) {
    PyErr_SetString(PyExc_OSError, "the library lacks an entry point of this binding");
    return nullptr;
  }
  Py_INCREF(err);
  Py_XSETREF(amq_error, err);
  api = found;
  Py_RETURN_NONE;
}

#define AMQ_METHOD(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"load", load, METH_VARARGS, nullptr},
    AMQ_METHOD(quantize_weights, 4), AMQ_METHOD(quantize_activations, 3), AMQ_METHOD(binary_gemm, 7),
    AMQ_METHOD(binary_gemv, 7), AMQ_METHOD(lstm_step, 15), AMQ_METHOD(lstm_step_static, 14),
    AMQ_METHOD(lstm_step_packed, 14), AMQ_METHOD(lstm_sequence, 14), AMQ_METHOD(gru_step, 14),
    AMQ_METHOD(gru_sequence, 14), AMQ_METHOD(embedding_lookup, 4), AMQ_METHOD(log_softmax, 2),
    AMQ_METHOD(softmax_layer, 9), AMQ_METHOD(lm_step, 20), AMQ_METHOD(lm_sequence, 20),
    AMQ_METHOD(lm_sequence_score, 21), AMQ_METHOD(dequantize, 4), AMQ_METHOD(fake_quantize, 3),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_amq_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__amq_torch(void) { return PyModule_Create(&module); }
