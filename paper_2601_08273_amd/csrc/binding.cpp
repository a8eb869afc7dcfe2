// The Python entry points' marshalling, in C++: what a call of the package does between its arguments and the C entry
// points of include/hippo.h -- the checks on the tensors, the descriptors, the outputs and workspaces that the caller did
// not pass, the current stream.  Nothing here computes.  The package's Python functions state the arguments, their defaults
// and the documentation, and make `stream` the current stream before they call in here.
//
// Why: the kernels of a small call take 8 to 20 us and so did its marshalling in Python, a tensor's attributes at 0.1 to
// 0.3 us each, an allocation at 2, a foreign call's conversions at 2.  us to issue, in Python -> here: a verification call
// with its buffers given 10 -> 7.3, of which its two launches 7; scoring 19.2 -> 12.9 (four launches), selection and
// gather 14.3 -> 6.9 (one, four outputs), the verdict 16.3 -> 8.9 (two).
//
// The library is reached through the addresses in the table below, which bind() looks up in the libhippo.so that the package
// loads.
#include <Python.h>
#include <dlfcn.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/ops/zeros.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <string>
#include <vector>

#include "hippo.h"

namespace {

#define HIPPO_LIBRARY(X)                                                                                              \
  X(hippo_workspace_bytes) X(hippo_score_layers_workspace_bytes) X(hippo_score_tokens_layers)     \
  X(hippo_select_gather_kv) X(hippo_verify_attention) X(hippo_draft_attention) X(hippo_verify_attention_append)         \
  X(hippo_draft_attention_append) X(hippo_verify_attention_paged) X(hippo_draft_attention_paged)                        \
  X(hippo_verify_attention_fp8kv) X(hippo_draft_attention_fp8kv) X(hippo_quantize_kv_workspace_bytes)                   \
  X(hippo_quantize_kv_e4m3) X(hippo_spec_verify_workspace_bytes) X(hippo_spec_verify)
struct Library {
#define X(name) decltype(&::name) name;
  HIPPO_LIBRARY(X)
#undef X
};
Library lib;
PyObject* video_desc_type;   // the package's VideoDesc, a ctypes structure laid out as hippo_video_desc
PyObject* hippo_error;       // the package's HippoError(status, what)

using at::Tensor;

// A Python exception is set; thrown through the entry point, which returns NULL for it.
struct Raised {};

void require(bool ok, const char* what) {
  if (ok) return;
  PyErr_SetString(PyExc_AssertionError, what);
  throw Raised();
}
#define REQUIRE(condition) require(condition, #condition)

void check(int status, const char* what) {
  if (status == HIPPO_OK) return;
  PyObject* e = PyObject_CallFunction(hippo_error, "is", status, what);
  if (e != nullptr) PyErr_SetObject(hippo_error, e);
  Py_XDECREF(e);
  throw Raised();
}

// A call of the library: other threads may run meanwhile, as during any foreign call.
template <typename Fn, typename... Args>
auto unlocked(Fn fn, Args... args) {
  PyThreadState* state = PyEval_SaveThread();
  const auto result = fn(args...);
  PyEval_RestoreThread(state);
  return result;
}

// ---- arguments ------------------------------------------------------------------------------------------------
const Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
    throw Raised();
  }
  return THPVariable_Unpack(o);
}
Tensor tensor_or_none(PyObject* o) { return o == Py_None ? Tensor() : tensor(o); }
long long integer(PyObject* o) {       // anything with __index__
  PyObject* i = PyNumber_Index(o);
  if (i == nullptr) throw Raised();
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(i);
  Py_DECREF(i);
  if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Raised();
  return (long long)v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Raised();
  return v != 0;
}
double number(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised();
  return v;
}
float scale_or_none(PyObject* o) { return o == Py_None ? 0.f : (float)number(o); }

hippo_video_desc video(PyObject* o) {
  if (!PyObject_TypeCheck(o, (PyTypeObject*)video_desc_type)) {
    PyErr_Format(PyExc_TypeError, "expected a VideoDesc, got %s", Py_TYPE(o)->tp_name);
    throw Raised();
  }
  Py_buffer view;
  if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw Raised();
  hippo_video_desc v;
  memcpy(&v, view.buf, sizeof v);
  PyBuffer_Release(&view);
  return v;
}
long long visual_tokens(const hippo_video_desc& v) { return (long long)v.n_frames * v.grid_h * v.grid_w; }

int dtype_code(const Tensor& t) {
  switch (t.scalar_type()) {
    case at::kFloat: return HIPPO_DTYPE_F32;
    case at::kBFloat16: return HIPPO_DTYPE_BF16;
    case at::kByte:
    case at::kFloat8_e4m3fn: return HIPPO_DTYPE_FP8_E4M3;      // E4M3 cache codes
    default: break;
  }
  PyErr_Format(PyExc_TypeError, "unsupported dtype %s (fp32, bf16, or uint8 / float8_e4m3fn cache codes)",
               c10::toString(t.scalar_type()));
  throw Raised();
}

// a [B, H_kv, N, d] cache, any strides with unit stride on d
hippo_kv_desc describe(const Tensor& cache, long long n_q_heads) {
  REQUIRE(cache.dim() == 4 && cache.stride(3) == 1);
  hippo_kv_desc d;
  d.batch = (int32_t)cache.size(0);
  d.n_q_heads = (int32_t)n_q_heads;
  d.n_kv_heads = (int32_t)cache.size(1);
  d.head_dim = (int32_t)cache.size(3);
  d.dtype = dtype_code(cache);
  d.stride_b = cache.stride(0);
  d.stride_h = cache.stride(1);
  d.stride_n = cache.stride(2);
  return d;
}
bool same_layout(const Tensor& a, const Tensor& b) { return a.sizes() == b.sizes() && a.strides() == b.strides(); }

template <typename T = void>
T* ptr(const Tensor& t) { return t.defined() ? (T*)t.data_ptr() : nullptr; }

Tensor empty(at::IntArrayRef sizes, at::ScalarType type, const Tensor& like) {
  return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}
// `given`, or a new one of nbytes() bytes
template <typename F>
Tensor workspace(PyObject* given, const Tensor& like, F nbytes) {
  if (given != Py_None) return tensor(given);
  return empty({std::max<long long>((long long)nbytes(), 256)}, at::kByte, like);
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

PyObject* none() { Py_RETURN_NONE; }
PyObject* wrap(const Tensor& t) { return t.defined() ? THPVariable_Wrap(t) : none(); }
PyObject* tuple(std::initializer_list<PyObject*> items) {      // takes the references
  PyObject* t = PyTuple_New((Py_ssize_t)items.size());
  Py_ssize_t i = 0;
  for (PyObject* o : items) PyTuple_SET_ITEM(t, i++, o);
  return t;
}

// ---- entry points: positional arguments, in the order of the package's functions without `stream` ----------------
PyObject* score(long long n_layers, const Tensor& q0, const Tensor& k0, const void* const* qs, const void* const* ks,
                long long emb_layer, PyObject* vid_o, PyObject* emb_o, PyObject* flags_o, PyObject* mass_o,
                PyObject* want_o, PyObject* scores_o, PyObject* ws_o, const char* what) {
  const hippo_kv_desc kv = describe(k0, q0.size(2));
  const hippo_video_desc vid = video(vid_o);
  const long long L = q0.size(1), n_vis = visual_tokens(vid);
  const uint32_t flags = (uint32_t)integer(flags_o);
  const Tensor emb = tensor_or_none(emb_o), mass = tensor_or_none(mass_o);
  long long emb_dim = 0, emb_stride = 0;
  if (emb.defined()) {
    REQUIRE(emb.dim() >= 3);
    emb_dim = emb.size(2);
    emb_stride = emb.stride(1);
    // What the kernels take for granted of embeddings that they read: the cache's type, channels side by side, batch elements
    // N_v tokens apart.  (The stride of a single element is nobody's: it may be cut from a longer sequence.  Elements beyond the
    // caches' are nobody's either.)
    if (!(flags & HIPPO_SCORE_ACCUMULATE_ONLY) && (flags & (HIPPO_SCORE_TEMP | HIPPO_SCORE_SPA))) {
      REQUIRE(emb.dim() == 3 && emb.stride(2) == 1 && emb.scalar_type() == k0.scalar_type());
      REQUIRE(emb.size(0) >= k0.size(0) && emb.size(1) >= n_vis);
      REQUIRE(k0.size(0) == 1 || emb.stride(0) == n_vis * emb.stride(1));
    }
  }
  const Tensor ws = workspace(ws_o, q0, [&] { return lib.hippo_score_layers_workspace_bytes(&kv, &vid, (int32_t)L, (int32_t)n_layers); });
  Tensor scores = tensor_or_none(scores_o), comps;
  if (!scores.defined() && !(flags & HIPPO_SCORE_ACCUMULATE_ONLY)) scores = empty({q0.size(0), n_vis}, at::kFloat, q0);
  const bool want = truth(want_o);
  if (want) comps = at::zeros({3, q0.size(0), n_vis}, at::TensorOptions().dtype(at::kFloat).device(q0.device()));
  check(unlocked(lib.hippo_score_tokens_layers, (int32_t)n_layers, qs, (int32_t)L, ks, (int32_t)emb_layer, &kv,
                 (int32_t)k0.size(2), &vid, ptr(emb), (int32_t)emb_dim, (int64_t)emb_stride, flags, ptr<float>(mass),
                 ptr<float>(scores), ptr<float>(comps), ptr(ws), (size_t)ws.numel(), stream()),
        what);
  return want ? tuple({wrap(scores), wrap(comps)}) : wrap(scores);
}

PyObject* score_tokens(PyObject* const* a) {
  const Tensor &q = tensor(a[0]), &k = tensor(a[1]);
  REQUIRE(q.is_contiguous() && q.dim() == 4);
  if (a[3] != Py_None) {
    const Tensor& emb = tensor(a[3]);
    REQUIRE(emb.dim() == 3 && emb.stride(2) == 1 && emb.stride(0) == emb.size(1) * emb.stride(1));
  }
  const void *qs = ptr(q), *ks = ptr(k);
  return score(1, q, k, &qs, &ks, 0, a[2], a[3], a[4], a[5], a[6], a[7], a[8], "hippo_score_tokens");
}

PyObject* score_tokens_layers(PyObject* const* a) {
  struct Items {                                               // the items of anything with a length and an index, while this
    PyObject* seq = nullptr;                                   // lives: a list, a tuple, the layers stacked in one tensor
    explicit Items(PyObject* o) {
      if (PyObject_Size(o) >= 0 && (PySequence_Check(o) || PyMapping_Check(o)))
        seq = PySequence_Fast(o, "expected one tensor per layer");
      if (seq != nullptr) return;
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "expected a list of tensors, one per layer");
      throw Raised();
    }
    ~Items() { Py_DECREF(seq); }
    Py_ssize_t size() const { return PySequence_Fast_GET_SIZE(seq); }
    const Tensor& operator[](Py_ssize_t i) const { return tensor(PySequence_Fast_GET_ITEM(seq, i)); }
  };
  const Items q(a[0]), k(a[1]);
  REQUIRE(q.size() == k.size() && q.size() >= 1);
  std::vector<const void*> qs, ks;
  for (Py_ssize_t i = 0; i < q.size(); ++i) {
    REQUIRE(q[i].is_contiguous() && q[i].sizes() == q[0].sizes() && same_layout(k[i], k[0]));
    qs.push_back(ptr(q[i]));
    ks.push_back(ptr(k[i]));
  }
  REQUIRE(q[0].dim() == 4);
  return score(q.size(), q[0], k[0], qs.data(), ks.data(), integer(a[3]), a[2], a[4], a[5], a[6], a[7], a[8], a[9],
               "hippo_score_tokens_layers");
}

// scores, k, k_src, v_src, vid, n_q_heads, gather, idx_out, k_dst, v_dst, workspace
PyObject* select_gather(PyObject* const* a) {
  const Tensor &scores = tensor(a[0]), &k_src = tensor(a[2]), &v_src = tensor(a[3]);
  const long long k = integer(a[1]);
  REQUIRE(scores.scalar_type() == at::kFloat && scores.is_contiguous());
  REQUIRE(k_src.dim() == 4 && same_layout(v_src, k_src));
  const hippo_video_desc vid = video(a[4]);
  const long long B = k_src.size(0), Hkv = k_src.size(1), N = k_src.size(2), d = k_src.size(3);
  long long H = a[5] == Py_None ? 0 : integer(a[5]);
  if (H == 0) H = Hkv;
  const hippo_kv_desc src = describe(k_src, H);
  hippo_kv_desc dst;
  Tensor idx = tensor_or_none(a[7]), k_dst, v_dst;
  if (!idx.defined()) idx = empty({B, k}, at::kInt, scores);
  const bool gather = truth(a[6]);
  if (gather) {
    const long long n_dst = N - visual_tokens(vid) + k;
    k_dst = tensor_or_none(a[8]);
    v_dst = tensor_or_none(a[9]);
    if (!k_dst.defined()) {
      k_dst = empty({B, Hkv, std::max<long long>(n_dst, 0), d}, k_src.scalar_type(), k_src);
      v_dst = at::empty_like(k_dst);
    }
    REQUIRE(k_dst.sizes() == at::IntArrayRef({B, Hkv, n_dst, d}) && v_dst.defined() && same_layout(v_dst, k_dst));
    dst = describe(k_dst, H);
  }
  const Tensor ws = workspace(a[10], scores, [] { return 256; });
  check(unlocked(lib.hippo_select_gather_kv, ptr<const float>(scores), (int32_t)k, ptr<const void>(k_src), ptr<const void>(v_src),
                 &src, (int32_t)N, &vid, ptr(k_dst), ptr(v_dst), gather ? &dst : nullptr, ptr<int32_t>(idx), ptr(ws),
                 (size_t)ws.numel(), stream()),
        "hippo_select_gather_kv");
  return tuple({wrap(idx), wrap(k_dst), wrap(v_dst)});
}

// what the attention calls have in common: q, the rows' statistics, the output, the workspace
struct AttentionCall {
  const Tensor& q;
  int call;
  long long ctx_len, num_splits;
  float scale;
  Tensor ws, out, lse;
  AttentionCall(PyObject* is_draft, PyObject* q_o, PyObject* ctx, PyObject* scale_o, PyObject* splits)
      : q(tensor(q_o)), call(truth(is_draft) ? HIPPO_CALL_DRAFT_ATTENTION : HIPPO_CALL_VERIFY_ATTENTION),
        ctx_len(integer(ctx)), num_splits(integer(splits)), scale(scale_or_none(scale_o)) {
    REQUIRE(q.is_contiguous() && q.dim() == 4);
  }
  bool draft() const { return call == HIPPO_CALL_DRAFT_ATTENTION; }
  int32_t q_len() const { return (int32_t)q.size(1); }
  void buffers(const hippo_kv_desc& kv, PyObject* want_lse, PyObject* out_o, PyObject* ws_o) {
    ws = workspace(ws_o, q, [&] {
      return lib.hippo_workspace_bytes(call, &kv, nullptr, q_len(), (int32_t)(ctx_len + q.size(1)), 0, (int32_t)num_splits);
    });
    out = out_o == Py_None ? at::empty_like(q) : tensor(out_o);
    if (truth(want_lse)) lse = empty({q.size(0), q.size(2), q.size(1)}, at::kFloat, q);
  }
  PyObject* result() const { return lse.defined() ? tuple({wrap(out), wrap(lse)}) : wrap(out); }
};

// draft, q, k_cache, v_cache, ctx_len, softmax_scale, num_splits, want_lse, out, workspace, k_new, v_new
PyObject* attention(PyObject* const* a) {
  AttentionCall c(a[0], a[1], a[4], a[5], a[6]);
  const Tensor &k = tensor(a[2]), &v = tensor(a[3]);
  const hippo_kv_desc kv = describe(k, c.q.size(2));
  REQUIRE(same_layout(v, k));
  c.buffers(kv, a[7], a[8], a[9]);
  if (a[10] != Py_None) {
    const Tensor &k_new = tensor(a[10]), &v_new = tensor(a[11]);
    const int64_t rows[4] = {c.q.size(0), c.q.size(1), k.size(1), c.q.size(3)};
    for (const Tensor* t : {&k_new, &v_new})
      REQUIRE(t->sizes() == at::IntArrayRef(rows) && t->is_contiguous() && t->scalar_type() == k.scalar_type());
    check(unlocked(c.draft() ? lib.hippo_draft_attention_append : lib.hippo_verify_attention_append, ptr<const void>(c.q),
                   c.q_len(), ptr<const void>(k_new), ptr<const void>(v_new), ptr(k), ptr(v), &kv, (int32_t)c.ctx_len, c.scale,
                   (int32_t)c.num_splits, ptr(c.out), ptr<float>(c.lse), ptr(c.ws), (size_t)c.ws.numel(), stream()),
          c.draft() ? "hippo_draft_attention_append" : "hippo_verify_attention_append");
  } else {
    check(unlocked(c.draft() ? lib.hippo_draft_attention : lib.hippo_verify_attention, ptr<const void>(c.q), c.q_len(),
                   ptr<const void>(k), ptr<const void>(v), &kv, (int32_t)c.ctx_len, c.scale, (int32_t)c.num_splits, ptr(c.out),
                   ptr<float>(c.lse), ptr(c.ws), (size_t)c.ws.numel(), stream()),
          c.draft() ? "hippo_draft_attention" : "hippo_verify_attention");
  }
  return c.result();
}

// draft, q, k_codes, v_codes, k_scale, v_scale, ctx_len, softmax_scale, num_splits, want_lse, out, workspace
PyObject* attention_fp8kv(PyObject* const* a) {
  AttentionCall c(a[0], a[1], a[6], a[7], a[8]);
  REQUIRE(c.q.scalar_type() == at::kBFloat16);
  const Tensor &k = tensor(a[2]), &v = tensor(a[3]), &ks = tensor(a[4]), &vs = tensor(a[5]);
  REQUIRE(k.dim() == 4 && k.stride(3) == 1 && dtype_code(k) == HIPPO_DTYPE_FP8_E4M3);
  REQUIRE(same_layout(v, k) && v.scalar_type() == k.scalar_type());
  for (const Tensor* t : {&ks, &vs})
    REQUIRE(t->sizes() == at::IntArrayRef({c.q.size(0), k.size(1)}) && t->is_contiguous() && t->scalar_type() == at::kFloat);
  hippo_kv_desc kv = describe(k, c.q.size(2));
  kv.batch = (int32_t)c.q.size(0);
  kv.head_dim = (int32_t)c.q.size(3);
  c.buffers(kv, a[9], a[10], a[11]);
  check(unlocked(c.draft() ? lib.hippo_draft_attention_fp8kv : lib.hippo_verify_attention_fp8kv, ptr<const void>(c.q), c.q_len(),
                 ptr<const void>(k), ptr<const void>(v), ptr<const float>(ks), ptr<const float>(vs), &kv, (int32_t)c.ctx_len,
                 c.scale, (int32_t)c.num_splits, ptr(c.out), ptr<float>(c.lse), ptr(c.ws), (size_t)c.ws.numel(), stream()),
        c.draft() ? "hippo_draft_attention_fp8kv" : "hippo_verify_attention_fp8kv");
  return c.result();
}

// draft, q, k_pool, v_pool, block_table, ctx_len, softmax_scale, num_splits, want_lse, out, workspace
PyObject* attention_paged(PyObject* const* a) {
  AttentionCall c(a[0], a[1], a[5], a[6], a[7]);
  const Tensor &k = tensor(a[2]), &v = tensor(a[3]), &table = tensor(a[4]);
  REQUIRE(k.dim() == 4 && k.stride(3) == 1);
  REQUIRE(same_layout(v, k));
  REQUIRE(table.scalar_type() == at::kInt && table.is_contiguous() && table.dim() >= 2 && table.size(0) == c.q.size(0));
  REQUIRE(table.numel() == table.size(0) * table.size(1));     // [B, max_pages], or with dimensions of 1 behind
  hippo_paged_kv_desc pd;
  pd.batch = (int32_t)c.q.size(0);
  pd.n_q_heads = (int32_t)c.q.size(2);
  pd.n_kv_heads = (int32_t)k.size(2);
  pd.head_dim = (int32_t)c.q.size(3);
  pd.dtype = dtype_code(k);
  pd.page_size = (int32_t)k.size(1);
  pd.max_pages = (int32_t)table.size(1);
  pd.n_pool_pages = (int32_t)k.size(0);
  pd.stride_page = k.stride(0);
  pd.stride_n = k.stride(1);
  pd.stride_h = k.stride(2);
  hippo_kv_desc flat;
  flat.batch = pd.batch;
  flat.n_q_heads = pd.n_q_heads;
  flat.n_kv_heads = pd.n_kv_heads;
  flat.head_dim = pd.head_dim;
  flat.dtype = pd.dtype;
  flat.stride_b = 0;
  flat.stride_h = pd.stride_h;
  flat.stride_n = pd.stride_n;
  c.buffers(flat, a[8], a[9], a[10]);
  check(unlocked(c.draft() ? lib.hippo_draft_attention_paged : lib.hippo_verify_attention_paged, ptr<const void>(c.q), c.q_len(),
                 ptr<const void>(k), ptr<const void>(v), ptr<const int32_t>(table), &pd, (int32_t)c.ctx_len, c.scale,
                 (int32_t)c.num_splits, ptr(c.out), ptr<float>(c.lse), ptr(c.ws), (size_t)c.ws.numel(), stream()),
        c.draft() ? "hippo_draft_attention_paged" : "hippo_verify_attention_paged");
  return c.result();
}

// k_src, v_src, n_rows, k_codes, v_codes, workspace
PyObject* quantize(PyObject* const* a) {
  const Tensor &k_src = tensor(a[0]), &v_src = tensor(a[1]);
  REQUIRE(k_src.dim() == 4);
  const long long B = k_src.size(0), Hkv = k_src.size(1), N = k_src.size(2), d = k_src.size(3);
  const long long n = a[2] == Py_None ? N : integer(a[2]);
  REQUIRE(same_layout(v_src, k_src) && 1 <= n && n <= N);
  const hippo_kv_desc src = describe(k_src, Hkv);
  Tensor k_codes = tensor_or_none(a[3]), v_codes = tensor_or_none(a[4]);
  if (!k_codes.defined()) {
    k_codes = empty({B, Hkv, n, d}, at::kByte, k_src);
    v_codes = at::empty_like(k_codes);
  }
  REQUIRE(k_codes.dim() == 4 && k_codes.size(0) == B && k_codes.size(1) == Hkv && k_codes.size(3) == d && k_codes.size(2) >= n);
  REQUIRE(v_codes.defined() && same_layout(v_codes, k_codes));
  const hippo_kv_desc dst = describe(k_codes, Hkv);
  const Tensor k_scale = empty({B, Hkv}, at::kFloat, k_src), v_scale = at::empty_like(k_scale);
  const Tensor ws = workspace(a[5], k_src, [&] { return lib.hippo_quantize_kv_workspace_bytes(&src, (int32_t)n); });
  check(unlocked(lib.hippo_quantize_kv_e4m3, ptr<const void>(k_src), ptr<const void>(v_src), &src, (int32_t)n, ptr(k_codes),
                 ptr(v_codes), &dst, ptr<float>(k_scale), ptr<float>(v_scale), ptr(ws), (size_t)ws.numel(), stream()),
        "hippo_quantize_kv_e4m3");
  return tuple({wrap(k_codes), wrap(v_codes), wrap(k_scale), wrap(v_scale)});
}

// p_logits, q_logits, draft_tokens, u_accept, u_sample, temperature, want_alpha, n_accept_out, next_token_out, workspace
PyObject* spec_verify(PyObject* const* a) {
  const Tensor& p = tensor(a[0]);
  REQUIRE(p.dim() == 3 && p.stride(2) == 1);
  const long long B = p.size(0), gamma = p.size(1) - 1, V = p.size(2);
  REQUIRE(B == 1 || p.stride(0) == p.size(1) * p.stride(1));
  Tensor q, tokens, u_accept;
  if (gamma != 0) {                                            // else nothing to verify: a plain draw from p_0
    q = tensor_or_none(a[1]);
    tokens = tensor_or_none(a[2]);
    u_accept = tensor_or_none(a[3]);
  }
  const Tensor u_sample = tensor_or_none(a[4]);
  long long q_stride = 0;
  if (q.defined()) {
    REQUIRE(q.sizes() == at::IntArrayRef({B, gamma, V}) && q.stride(2) == 1 && q.scalar_type() == p.scalar_type());
    REQUIRE(B == 1 || q.stride(0) == gamma * q.stride(1));
    q_stride = q.stride(1);
  }
  REQUIRE(!tokens.defined() || (tokens.scalar_type() == at::kInt && tokens.is_contiguous()));
  REQUIRE(!u_accept.defined() || (u_accept.scalar_type() == at::kFloat && u_accept.is_contiguous()));
  REQUIRE(!u_sample.defined() || (u_sample.scalar_type() == at::kFloat && u_sample.is_contiguous()));
  const float temperature = (float)number(a[5]);
  const bool want = truth(a[6]);
  Tensor n_acc = tensor_or_none(a[7]), next = tensor_or_none(a[8]), alpha;
  if (!n_acc.defined()) n_acc = empty({B}, at::kInt, p);
  if (!next.defined()) next = empty({B}, at::kInt, p);
  if (want) alpha = empty({B, gamma}, at::kFloat, p);
  const int code = dtype_code(p);
  const Tensor ws = workspace(a[9], p, [&] {
    return lib.hippo_spec_verify_workspace_bytes((int32_t)B, (int32_t)gamma, (int32_t)V, code);
  });
  check(unlocked(lib.hippo_spec_verify, ptr<const void>(p), ptr<const void>(q), code, (int64_t)p.stride(1), (int64_t)q_stride,
                 ptr<const int32_t>(tokens), ptr<const float>(u_accept), ptr<const float>(u_sample), (int32_t)B, (int32_t)gamma,
                 (int32_t)V, temperature, ptr<int32_t>(n_acc), ptr<int32_t>(next), ptr<float>(alpha), ptr(ws),
                 (size_t)ws.numel(), stream()),
        "hippo_spec_verify");
  return want ? tuple({wrap(n_acc), wrap(next), wrap(alpha)}) : tuple({wrap(n_acc), wrap(next)});
}

// bind(path of libhippo.so, VideoDesc, HippoError)
PyObject* bind(PyObject* const* a) {
  const char* path = PyUnicode_AsUTF8(a[0]);
  if (path == nullptr) throw Raised();
  void* handle = dlopen(path, RTLD_NOW | RTLD_LOCAL);          // (the package keeps it loaded)
  if (handle == nullptr) {
    PyErr_SetString(PyExc_RuntimeError, dlerror());
    throw Raised();
  }
  Library found;
#define X(name)                                                                   \
  found.name = (decltype(&::name))dlsym(handle, #name);                           \
  if (found.name == nullptr) {                                                    \
    PyErr_SetString(PyExc_RuntimeError, "libhippo.so has no " #name);             \
    throw Raised();                                                               \
  }
  HIPPO_LIBRARY(X)
#undef X
  lib = found;
  Py_INCREF(a[1]);
  Py_XSETREF(video_desc_type, a[1]);
  Py_INCREF(a[2]);
  Py_XSETREF(hippo_error, a[2]);
  return none();
}

template <PyObject* (*F)(PyObject* const*), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != N) {
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", N, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

#define ENTRY(name, n) {#name, (PyCFunction)(void (*)(void))entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    ENTRY(bind, 3), ENTRY(score_tokens, 9), ENTRY(score_tokens_layers, 10), ENTRY(select_gather, 11), ENTRY(attention, 12),
    ENTRY(attention_fp8kv, 12), ENTRY(attention_paged, 11), ENTRY(quantize, 6), ENTRY(spec_verify, 10), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module_def); }
