// Native argument checks and marshalling of the Python binding's serving-loop
// calls: a call that hands over every buffer (outputs and workspace) goes from
// its tensors to the C ABI without interpreted code in between.  In Python
// the checks, the dims struct and the pointer conversions of a call took
// 10-15 us, as long as or longer than the kernels of a small launch (one
// layer's attention over one sequence: 11.5 us of kernels, 17.9 us a call).
//
// Every function takes what its Python wrapper takes, checks what the wrapper
// checks (and that the caller's buffers have the documented form) and returns
//   None  when anything is not as expected: nothing has been done, and the
//         wrapper goes on with its own checks, which raise what is wrong or
//         accept what is merely unusual (tensor subclasses, tracing and
//         batching wrappers, other output layouts);
//   int   the status of the C entry point otherwise.
// No tensor, pointer or result is kept from one call to the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/spec.h"

namespace {

// The C entry points, set once by init() from the loaded library.
struct Api {
  decltype(&spec_score) score;
  decltype(&spec_topk) topk;
  decltype(&spec_sparse_decode_attn) attn;
  decltype(&spec_step) step;
  decltype(&spec_retrieval_qk) retrieval_qk;
  decltype(&spec_mla_sparse_decode_attn) mla;
};
Api api = {};

// A plain device tensor: torch.Tensor or Parameter itself, whose dispatch
// beneath autograd and autocast is the device's own (no subclass, fake,
// batched, functional or other wrapper), with memory.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckTypeExact(Py_TYPE(o))) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || !t.has_storage()) return nullptr;
  const c10::DispatchKeySet under =
      t.key_set() - c10::autograd_dispatch_keyset_with_ADInplaceOrView -
      c10::autocast_dispatch_keyset;
  if (under.highestPriorityTypeId() != c10::DispatchKey::CUDA) return nullptr;
  return &t;
}

bool is(const at::Tensor* t, at::ScalarType type, int64_t ndim) {
  return t && t->scalar_type() == type && t->dim() == ndim;
}

// The last n dims are densely packed (row-major).
bool packed(const at::Tensor& t, int64_t n) {
  int64_t expect = 1;
  for (int64_t d = t.dim() - 1; d >= t.dim() - n; --d) {
    if (t.size(d) != 1 && t.stride(d) != expect) return false;
    expect *= t.size(d);
  }
  return true;
}

bool has_shape(const at::Tensor* t, at::ScalarType type, std::initializer_list<int64_t> shape) {
  return t && t->scalar_type() == type && t->is_contiguous() &&
         t->sizes() == c10::IntArrayRef(shape.begin(), shape.size());
}

bool same_device(const at::Tensor& a, std::initializer_list<const at::Tensor*> others) {
  for (const at::Tensor* t : others)
    if (t && t->device() != a.device()) return false;
  return true;
}

template <class T>
T* ptr(const at::Tensor* t) {
  return t ? static_cast<T*>(t->data_ptr()) : nullptr;
}

bool as_int(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long x = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}

bool as_float(PyObject* o, float* v) {
  if (!PyFloat_CheckExact(o)) return false;
  *v = (float)PyFloat_AS_DOUBLE(o);
  return true;
}

void* as_stream(PyObject* o, bool* ok) {
  *ok = PyLong_CheckExact(o);
  return *ok ? PyLong_AsVoidPtr(o) : nullptr;
}

spec_dims base_dims() {
  spec_dims d = {};
  d.H_r = 8;
  d.d_r = 64;
  d.n_layers = 1;
  d.H_q = 1;
  d.H_kv = 1;
  d.d = 128;
  d.n_sets = 1;
  return d;
}

// K and V caches of one shape and layout, the inner [token][head][dim] block dense.
bool caches(const at::Tensor* K, const at::Tensor* V) {
  return is(K, at::kBFloat16, 5) && is(V, at::kBFloat16, 5) && K->sizes() == V->sizes() &&
         K->strides() == V->strides() && packed(*K, 3);
}

#define TENSOR(name, i)                       \
  const at::Tensor* name = plain(args[i]);    \
  if (!name) Py_RETURN_NONE
#define TENSOR_OR_NONE(name, i)                                  \
  const at::Tensor* name = nullptr;                              \
  if (args[i] != Py_None && !(name = plain(args[i]))) Py_RETURN_NONE
#define EXPECT(x) \
  if (!(x)) Py_RETURN_NONE

// Calls f without the GIL.  The arguments, the tensors' pointers among them, are
// evaluated by the caller, so no tensor is touched while other threads run; an
// exception finds the GIL held again.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

template <class F, class... A>
PyObject* call(F f, A... args) {
  spec_status st;
  {
    Unlocked unlocked;
    st = f(args...);
  }
  return PyLong_FromLong((long)st);
}

// attn(q, K, V, counts, idx|None, scale, out, lse|None, ws, stream)
PyObject* fast_attn(PyObject*, PyObject* const* args, Py_ssize_t n) {
  EXPECT(n == 10);
  TENSOR(q, 0);
  TENSOR(K, 1);
  TENSOR(V, 2);
  TENSOR(counts, 3);
  TENSOR_OR_NONE(idx, 4);
  TENSOR(out, 6);
  TENSOR_OR_NONE(lse, 7);
  TENSOR(ws, 8);
  spec_dims d = base_dims();
  bool ok;
  EXPECT(as_float(args[5], &d.scale));
  void* stream = as_stream(args[9], &ok);
  EXPECT(ok && is(q, at::kBFloat16, 4) && q->is_contiguous() && caches(K, V));
  const int64_t nl = K->size(0), B = K->size(1), L = K->size(2), H_kv = K->size(3),
                hd = K->size(4), H_q = q->size(2);
  EXPECT(q->size(0) == nl && q->size(1) == B && q->size(3) == hd);
  EXPECT(has_shape(counts, at::kInt, {B}));
  int64_t k_max = L;
  if (idx) {
    EXPECT(idx->scalar_type() == at::kInt && idx->is_contiguous());
    EXPECT(idx->dim() == 2 || (idx->dim() == 3 && idx->size(1) == H_kv));
    EXPECT(idx->size(0) == B);
    d.n_sets = idx->dim() == 3 ? (int32_t)H_kv : 1;
    k_max = idx->size(-1);
  } else {
    EXPECT(K->is_contiguous());
  }
  EXPECT(has_shape(out, at::kFloat, {nl, B, H_q, hd}));
  EXPECT(!lse || has_shape(lse, at::kFloat, {nl, B, H_q}));
  EXPECT(same_device(*q, {K, V, counts, idx, out, lse, ws}));
  d.B = (int32_t)B;
  d.L_cap = d.L_max = (int32_t)L;
  d.k_max = (int32_t)k_max;
  d.n_layers = (int32_t)nl;
  d.H_q = (int32_t)H_q;
  d.H_kv = (int32_t)H_kv;
  d.d = (int32_t)hd;
  d.kv_stride_layer = K->stride(0);
  d.kv_stride_b = K->stride(1);
  return call(api.attn, &d, ptr<uint16_t>(q), ptr<uint16_t>(K), ptr<uint16_t>(V), ptr<int32_t>(idx),
              ptr<int32_t>(counts), ptr<float>(out), ptr<float>(lse), ws->data_ptr(),
              ws->nbytes(), stream);
}

// score(q_r, K_r, seq_lens, L_max|None, scale_r, out, ws, n_sets, stream)
PyObject* fast_score(PyObject*, PyObject* const* args, Py_ssize_t n) {
  EXPECT(n == 9);
  TENSOR(q_r, 0);
  TENSOR(K_r, 1);
  TENSOR(seq_lens, 2);
  TENSOR(out, 5);
  TENSOR(ws, 6);
  spec_dims d = base_dims();
  bool ok;
  int32_t n_sets;
  EXPECT(as_float(args[4], &d.scale_r) && as_int(args[7], &n_sets));
  void* stream = as_stream(args[8], &ok);
  EXPECT(ok && is(K_r, at::kBFloat16, 4) && packed(*K_r, 3));
  const int64_t B = K_r->size(0), L_cap = K_r->size(1), H_r = K_r->size(2), d_r = K_r->size(3);
  EXPECT(has_shape(q_r, at::kBFloat16, {B, H_r, d_r}) && has_shape(seq_lens, at::kInt, {B}));
  int32_t L_max = (int32_t)L_cap;
  EXPECT(args[3] == Py_None || as_int(args[3], &L_max));
  if (n_sets == 1) {
    EXPECT(has_shape(out, at::kFloat, {B, L_max}));
  } else {
    EXPECT(has_shape(out, at::kFloat, {B, n_sets, L_max}));
  }
  EXPECT(same_device(*K_r, {q_r, seq_lens, out, ws}));
  d.B = (int32_t)B;
  d.L_cap = (int32_t)L_cap;
  d.L_max = L_max;
  d.k_max = 1;
  d.H_r = (int32_t)H_r;
  d.d_r = (int32_t)d_r;
  d.H_q = d.H_kv = d.n_sets = n_sets;
  d.kr_stride_b = K_r->stride(0);
  return call(api.score, &d, ptr<uint16_t>(q_r), ptr<uint16_t>(K_r), ptr<int32_t>(seq_lens),
              ptr<float>(out), ws->data_ptr(), ws->nbytes(), stream);
}

// topk(scores, seq_lens, ks, k_max, idx, counts, ws, stream)
PyObject* fast_topk(PyObject*, PyObject* const* args, Py_ssize_t n) {
  EXPECT(n == 8);
  TENSOR(scores, 0);
  TENSOR(seq_lens, 1);
  TENSOR(ks, 2);
  TENSOR(idx, 4);
  TENSOR(counts, 5);
  TENSOR(ws, 6);
  spec_dims d = base_dims();
  bool ok;
  EXPECT(as_int(args[3], &d.k_max));
  void* stream = as_stream(args[7], &ok);
  EXPECT(ok && scores->scalar_type() == at::kFloat && scores->is_contiguous());
  EXPECT(scores->dim() == 2 || scores->dim() == 3);
  const int64_t B = scores->size(0), L = scores->size(-1);
  const int64_t n_sets = scores->dim() == 3 ? scores->size(1) : 1;
  EXPECT(has_shape(seq_lens, at::kInt, {B}) && has_shape(ks, at::kInt, {B}) &&
         has_shape(counts, at::kInt, {B}));
  if (scores->dim() == 2) {
    EXPECT(has_shape(idx, at::kInt, {B, d.k_max}));
  } else {
    EXPECT(has_shape(idx, at::kInt, {B, n_sets, d.k_max}));
  }
  EXPECT(same_device(*scores, {seq_lens, ks, idx, counts, ws}));
  d.B = (int32_t)B;
  d.L_cap = d.L_max = (int32_t)L;
  d.H_q = d.H_kv = d.n_sets = (int32_t)n_sets;
  return call(api.topk, &d, ptr<float>(scores), ptr<int32_t>(seq_lens), ptr<int32_t>(ks),
              ptr<int32_t>(idx), ptr<int32_t>(counts), ws->data_ptr(), ws->nbytes(), stream);
}

// step(q_r, K_r, seq_lens, ks, q, K, V, k_max, L_max|None, scale_r, scale,
//      elastic's (slot_tok, kbuf, vbuf, n_changed, slot_src)|None, outputs,
//      head_level, ws, stream)
PyObject* fast_step(PyObject*, PyObject* const* args, Py_ssize_t n) {
  EXPECT(n == 16);
  TENSOR(q_r, 0);
  TENSOR(K_r, 1);
  TENSOR(seq_lens, 2);
  TENSOR(ks, 3);
  TENSOR(q, 4);
  TENSOR(K, 5);
  TENSOR(V, 6);
  TENSOR(ws, 14);
  spec_dims d = base_dims();
  bool ok;
  EXPECT(as_int(args[7], &d.k_max) && as_float(args[9], &d.scale_r) &&
         as_float(args[10], &d.scale) && PyBool_Check(args[13]) && PyDict_CheckExact(args[12]));
  void* stream = as_stream(args[15], &ok);
  EXPECT(ok && is(K_r, at::kBFloat16, 4) && packed(*K_r, 3) && caches(K, V));
  const int64_t nl = K->size(0), B = K->size(1), H_kv = K->size(3), hd = K->size(4);
  const int64_t H_r = K_r->size(2), d_r = K_r->size(3);
  EXPECT(K_r->size(0) == B && has_shape(q_r, at::kBFloat16, {B, H_r, d_r}));
  EXPECT(is(q, at::kBFloat16, 4) && q->is_contiguous() && q->size(0) == nl && q->size(1) == B &&
         q->size(3) == hd);
  const int64_t H_q = q->size(2);
  EXPECT(has_shape(seq_lens, at::kInt, {B}) && has_shape(ks, at::kInt, {B}));
  const int64_t L_cap = std::min(K_r->size(1), K->size(2));
  d.L_cap = (int32_t)L_cap;
  d.L_max = (int32_t)L_cap;
  EXPECT(args[8] == Py_None || as_int(args[8], &d.L_max));

  PyObject* o = args[12];
  const at::Tensor* outs[5];  // idx, counts, out, lse, scores
  static const char* const names[5] = {"idx", "counts", "out", "lse", "scores"};
  for (int i = 0; i < 5; ++i) {
    PyObject* v = PyDict_GetItemString(o, names[i]);  // borrowed
    outs[i] = nullptr;
    if (!v || v == Py_None) {
      EXPECT(i >= 3);
      continue;
    }
    EXPECT((outs[i] = plain(v)) != nullptr);
  }
  const bool sets = args[13] == Py_True;
  if (sets) {
    EXPECT(has_shape(outs[0], at::kInt, {B, H_kv, d.k_max}));
    EXPECT(!outs[4] || has_shape(outs[4], at::kFloat, {B, H_kv, d.L_max}));
  } else {
    EXPECT(has_shape(outs[0], at::kInt, {B, d.k_max}));
    EXPECT(!outs[4] || has_shape(outs[4], at::kFloat, {B, d.L_max}));
  }
  EXPECT(has_shape(outs[1], at::kInt, {B}) && has_shape(outs[2], at::kFloat, {nl, B, H_q, hd}));
  EXPECT(!outs[3] || has_shape(outs[3], at::kFloat, {nl, B, H_q}));
  EXPECT(same_device(*q, {q_r, K_r, seq_lens, ks, K, V, ws, outs[0], outs[1], outs[2], outs[3],
                          outs[4]}));

  spec_elastic el = {};
  const bool elastic = args[11] != Py_None;
  if (elastic) {
    EXPECT(PyTuple_CheckExact(args[11]) && PyTuple_GET_SIZE(args[11]) == 5);
    const at::Tensor* e[5];
    for (int i = 0; i < 5; ++i) EXPECT((e[i] = plain(PyTuple_GET_ITEM(args[11], i))) != nullptr);
    for (int i : {0, 4}) EXPECT(has_shape(e[i], at::kInt, {B, d.k_max}));
    for (int i : {1, 2}) EXPECT(has_shape(e[i], at::kBFloat16, {nl, B, d.k_max, H_kv, hd}));
    EXPECT(has_shape(e[3], at::kInt, {B}) && same_device(*q, {e[0], e[1], e[2], e[3], e[4]}));
    el = {ptr<int32_t>(e[0]), ptr<uint16_t>(e[1]), ptr<uint16_t>(e[2]), ptr<int32_t>(e[3]),
          ptr<int32_t>(e[4])};
  }
  d.B = (int32_t)B;
  d.H_r = (int32_t)H_r;
  d.d_r = (int32_t)d_r;
  d.n_layers = (int32_t)nl;
  d.H_q = (int32_t)H_q;
  d.H_kv = (int32_t)H_kv;
  d.d = (int32_t)hd;
  d.kr_stride_b = K_r->stride(0);
  d.kv_stride_layer = K->stride(0);
  d.kv_stride_b = K->stride(1);
  d.n_sets = sets ? (int32_t)H_kv : 1;
  return call(api.step, &d, ptr<uint16_t>(q_r), ptr<uint16_t>(K_r), ptr<int32_t>(seq_lens),
              ptr<int32_t>(ks), ptr<uint16_t>(q), ptr<uint16_t>(K), ptr<uint16_t>(V),
              ptr<int32_t>(outs[0]), ptr<int32_t>(outs[1]), ptr<float>(outs[2]),
              ptr<float>(outs[3]), ptr<float>(outs[4]), elastic ? &el : nullptr, ws->data_ptr(),
              ws->nbytes(), stream);
}

// retrieval_qk(tokens, pos, emb, w_q, w_k, K_r, rope_base, yarn_scale,
//              yarn_orig_ctx, yarn_alpha, yarn_beta, q_r, ws, stream)
PyObject* fast_retrieval_qk(PyObject*, PyObject* const* args, Py_ssize_t n) {
  EXPECT(n == 14);
  TENSOR(tokens, 0);
  TENSOR(pos, 1);
  TENSOR(emb, 2);
  TENSOR(w_q, 3);
  TENSOR(w_k, 4);
  TENSOR(K_r, 5);
  TENSOR(q_r, 11);
  TENSOR(ws, 12);
  spec_frontend fe = {};
  bool ok;
  EXPECT(as_float(args[6], &fe.rope_base) && as_float(args[7], &fe.yarn_scale) &&
         as_int(args[8], &fe.yarn_orig_ctx) && as_float(args[9], &fe.yarn_alpha) &&
         as_float(args[10], &fe.yarn_beta));
  void* stream = as_stream(args[13], &ok);
  EXPECT(ok && is(K_r, at::kBFloat16, 4) && packed(*K_r, 3));
  const int64_t B = K_r->size(0), L = K_r->size(1), H_r = K_r->size(2), d_r = K_r->size(3);
  EXPECT(has_shape(tokens, at::kInt, {B}) && has_shape(pos, at::kInt, {B}));
  EXPECT(is(emb, at::kBFloat16, 2) && emb->is_contiguous());
  const int64_t hidden = emb->size(1);
  EXPECT(has_shape(w_q, at::kBFloat16, {H_r * d_r, hidden}) &&
         has_shape(w_k, at::kBFloat16, {H_r * d_r, hidden}) &&
         has_shape(q_r, at::kBFloat16, {B, H_r, d_r}));
  EXPECT(same_device(*K_r, {tokens, pos, emb, w_q, w_k, q_r, ws}));
  spec_dims d = base_dims();
  d.B = (int32_t)B;
  d.L_cap = d.L_max = (int32_t)L;
  d.k_max = 1;
  d.H_r = (int32_t)H_r;
  d.d_r = (int32_t)d_r;
  d.kr_stride_b = K_r->stride(0);
  fe.vocab = (int32_t)emb->size(0);
  fe.hidden = (int32_t)hidden;
  return call(api.retrieval_qk, &d, &fe, ptr<int32_t>(tokens), ptr<int32_t>(pos),
              ptr<uint16_t>(emb), ptr<uint16_t>(w_q), ptr<uint16_t>(w_k), ptr<uint16_t>(q_r),
              ptr<uint16_t>(K_r), ws->data_ptr(), ws->nbytes(), stream);
}

// mla(q, ckv, w_uk, w_uv, idx, counts, scale, out, lse|None, ws, stream)
PyObject* fast_mla(PyObject*, PyObject* const* args, Py_ssize_t n) {
  EXPECT(n == 11);
  TENSOR(q, 0);
  TENSOR(ckv, 1);
  TENSOR(w_uk, 2);
  TENSOR(w_uv, 3);
  TENSOR(idx, 4);
  TENSOR(counts, 5);
  TENSOR(out, 7);
  TENSOR_OR_NONE(lse, 8);
  TENSOR(ws, 9);
  spec_mla_dims d = {};
  bool ok;
  EXPECT(as_float(args[6], &d.scale));
  void* stream = as_stream(args[10], &ok);
  EXPECT(ok && is(ckv, at::kBFloat16, 4) && packed(*ckv, 2) && is(w_uk, at::kBFloat16, 4) &&
         is(w_uv, at::kBFloat16, 4) && is(q, at::kBFloat16, 4));
  const int64_t nl = ckv->size(0), B = ckv->size(1), L = ckv->size(2), H = q->size(2),
                dn = w_uk->size(2), dc = w_uk->size(3), dv = w_uv->size(2),
                dr = ckv->size(3) - dc;
  EXPECT(has_shape(q, at::kBFloat16, {nl, B, H, dn + dr}) &&
         has_shape(w_uk, at::kBFloat16, {nl, H, dn, dc}) &&
         has_shape(w_uv, at::kBFloat16, {nl, H, dv, dc}));
  EXPECT(is(idx, at::kInt, 2) && idx->is_contiguous() && idx->size(0) == B);
  EXPECT(has_shape(counts, at::kInt, {B}) && has_shape(out, at::kFloat, {nl, B, H, dv}));
  EXPECT(!lse || has_shape(lse, at::kFloat, {nl, B, H}));
  EXPECT(same_device(*q, {ckv, w_uk, w_uv, idx, counts, out, lse, ws}));
  d.B = (int32_t)B;
  d.L_cap = (int32_t)L;
  d.k_max = (int32_t)idx->size(1);
  d.n_layers = (int32_t)nl;
  d.H = (int32_t)H;
  d.d_c = (int32_t)dc;
  d.d_rope = (int32_t)dr;
  d.d_nope = (int32_t)dn;
  d.d_v = (int32_t)dv;
  d.ckv_stride_layer = ckv->stride(0);
  d.ckv_stride_b = ckv->stride(1);
  return call(api.mla, &d, ptr<uint16_t>(q), ptr<uint16_t>(ckv), ptr<uint16_t>(w_uk),
              ptr<uint16_t>(w_uv), ptr<int32_t>(idx), ptr<int32_t>(counts), ptr<float>(out),
              ptr<float>(lse), ws->data_ptr(), ws->nbytes(), stream);
}

// init(addresses of the entry points, in Api's order)
PyObject* fast_init(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != (Py_ssize_t)(sizeof(Api) / sizeof(void*))) {
    PyErr_SetString(PyExc_TypeError, "init: one address per entry point");
    return nullptr;
  }
  void* a[sizeof(Api) / sizeof(void*)];
  for (Py_ssize_t i = 0; i < n; ++i) {
    a[i] = PyLong_AsVoidPtr(args[i]);
    if (!a[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "init: null address");
      return nullptr;
    }
  }
  memcpy(&api, a, sizeof(api));
  Py_RETURN_NONE;
}

// C++ exceptions (torch's checks) leave as the wrapper's own path: None.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  try {
    if (F != fast_init && !api.step) Py_RETURN_NONE;
    return F(self, args, n);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

#define METHOD(name, f)                                                                   \
  {                                                                                       \
    name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(guarded<f>)),    \
        METH_FASTCALL, nullptr                                                            \
  }
PyMethodDef methods[] = {
    METHOD("init", fast_init),
    METHOD("attn", fast_attn),
    METHOD("score", fast_score),
    METHOD("topk", fast_topk),
    METHOD("step", fast_step),
    METHOD("retrieval_qk", fast_retrieval_qk),
    METHOD("mla", fast_mla),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__fast(void) { return PyModule_Create(&module); }
