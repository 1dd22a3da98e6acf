// Argument marshalling of the Python binding in native code: the per-call part of decode, prefill, append, compress and
// re-compress.  What a call on a small cache costs is mostly this part: in Python with ctypes a decode call of 7 us of
// kernels took 13.3 us (8 data_ptr() calls and a ctypes structure for the cache, three allocations, two library calls) and takes
// 9 here, compressing 2K tokens 16.1 and 8.5.
//
// Every function repeats the binding's checks and returns None for a call that fails one or that it does not take as it is (other
// types than exact tensors, a number that is neither int nor float); the binding's Python code then takes it, so which error a
// refused call raises is written down there only.  Nothing is kept between calls but the types and the library's entry points.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/Context.h>
#include <ATen/hip/EmptyTensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/record_function.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "hs.h"

namespace {

struct Entries {  // of libhs.so, as the binding has loaded it
  decltype(&hs_kv_bytes) kv_bytes;
  decltype(&hs_workspace_bytes) workspace_bytes;
  decltype(&hs_decode_auto_splits) auto_splits;
  decltype(&hs_decode_attn) decode;
  decltype(&hs_decode_attn_static) decode_static;
  decltype(&hs_decode_attn_tail) decode_tail;
  decltype(&hs_decode_attn_tail_rows) decode_tail_rows;
  decltype(&hs_prefill_plan) prefill_plan;
  decltype(&hs_prefill_attn_ws) prefill;
  decltype(&hs_append_tiles) append;
  decltype(&hs_append_tile_rows) append_rows;
  decltype(&hs_tile_counts) tile_counts;
  decltype(&hs_compress_kv) compress;
  decltype(&hs_recompress_kv) recompress;
} g_hs;
PyTypeObject *g_shape_type, *g_policy_type, *g_kv_type;

enum { S_K_DENSE, S_K_NNZ, S_K_META, S_K_MAP, S_V_DENSE, S_V_NNZ, S_V_META, S_V_MAP, S_COUNTS, S_UNIFORM, N_NAMES };
const char* const kNames[N_NAMES] = {"k_dense", "k_nnz", "k_meta", "k_map", "v_dense", "v_nnz", "v_meta", "v_map", "counts", "uniform"};
PyObject* g_names[N_NAMES];

bool exact_tensor(PyObject* o) { return THPVariable_CheckExact(o); }
bool none_or_tensor(PyObject* o) { return o == Py_None || exact_tensor(o); }
const at::Tensor& tensor(PyObject* o) { return THPVariable_Unpack(o); }
void* address(PyObject* o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }

bool get_int(PyObject* o, int32_t* v) {  // a Python int in range; bool is one
  if (!PyLong_Check(o)) return false;
  int over = 0;
  const long x = PyLong_AsLongAndOverflow(o, &over);
  if (over != 0 || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}
bool get_float(PyObject* o, float* v) {
  if (PyFloat_Check(o)) { *v = (float)PyFloat_AS_DOUBLE(o); return true; }
  int32_t i;
  if (!get_int(o, &i)) return false;
  *v = (float)i;
  return true;
}

bool get_struct(PyObject* o, PyTypeObject* type, void* s, size_t size) {  // the bytes of one of the binding's ctypes structures
  if (Py_TYPE(o) != type) return false;
  Py_buffer b;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return false; }
  const bool ok = b.len == (Py_ssize_t)size;
  if (ok) memcpy(s, b.buf, size);
  PyBuffer_Release(&b);
  return ok;
}
bool get_shape(PyObject* o, hs_shape* s) { return get_struct(o, g_shape_type, s, sizeof(*s)); }
bool get_policy(PyObject* o, hs_policy* p) { return get_struct(o, g_policy_type, p, sizeof(*p)); }
bool get_counts(PyObject* o, int32_t c[5]) {
  if (!PyList_CheckExact(o) || PyList_GET_SIZE(o) != 5) return false;
  for (int i = 0; i < 5; i++)
    if (!get_int(PyList_GET_ITEM(o, i), &c[i])) return false;
  return true;
}

// the cache's buffers as the object holds them now
bool get_kv(PyObject* o, hs_kv* kv) {
  if (Py_TYPE(o) != g_kv_type) return false;
  void** ptr[8] = {&kv->k_dense, &kv->k_nnz, &kv->k_meta, (void**)&kv->k_map, &kv->v_dense, &kv->v_nnz, &kv->v_meta, (void**)&kv->v_map};
  bool ok = true;
  for (int i = 0; i < N_NAMES && ok; i++) {
    PyObject* a = PyObject_GetAttr(o, g_names[i]);
    if (a == nullptr) { PyErr_Clear(); return false; }
    if (i < 8) {
      ok = none_or_tensor(a);
      if (ok) *ptr[i] = address(a);  // the object keeps the tensor alive
    } else if (i == S_COUNTS) {
      ok = PyList_CheckExact(a) && PyList_GET_SIZE(a) >= 5 && get_int(PyList_GET_ITEM(a, 1), &kv->cap_dense_k) &&
           get_int(PyList_GET_ITEM(a, 2), &kv->cap_sparse_k) && get_int(PyList_GET_ITEM(a, 3), &kv->cap_dense_v) &&
           get_int(PyList_GET_ITEM(a, 4), &kv->cap_sparse_v);
    } else {
      ok = get_int(a, &kv->uniform);
    }
    Py_DECREF(a);
  }
  return ok;
}

at::ScalarType element_type(const hs_shape& s) { return s.dtype == HS_FP16 ? at::kHalf : at::kBFloat16; }
bool query_ok(const at::Tensor& q, const hs_shape& s) { return q.scalar_type() == element_type(s) && q.is_contiguous() && q.is_cuda(); }
void* current_stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// New tensors on the device of `like`.  A call on a small cache is mostly its allocations (two to nine), and a third of one is the
// dispatcher's two rounds, so where these have nothing to do the tensor is made by what they end in: not where anything listens
// to the operators of this thread (dispatch modes, fake tensors, function transforms, profilers and other observers) or new memory is to be
// filled.  Looking that up is for calls that make a tensor: those into kept buffers go without.
// us a call through the dispatcher / at once, 1K tokens: decode with outputs and scratch of its own 9.9 / 9.3, prefill 6.1 / 5.7, compress
// 10.2 / 8.4, re-compress 11.3 / 9.7; of that, asking for observers is 0.01 to 0.04.
class NewTensors {
 public:
  explicit NewTensors(const at::Tensor& like) : like_(like) {
    const auto usual = c10::DispatchKeySet({c10::DispatchKey::BackendSelect, c10::DispatchKey::ADInplaceOrView});
    const auto& context = at::globalContext();
    at_once_ = (c10::impl::tls_local_dispatch_key_set().included_ - usual).empty() && like.is_cuda() && !at::hasCallbacks() &&
               !(context.deterministicAlgorithms() && context.deterministicFillUninitializedMemory());
  }
  at::Tensor operator()(at::IntArrayRef sizes, at::ScalarType type) const {
    if (!at_once_) return at::empty(sizes, like_.options().dtype(type));
    return at::Tensor(at::detail::empty_cuda(sizes, type, like_.device(), std::nullopt));
  }
  at::Tensor beside() const {  // of the sizes, strides and type of `like`, which is contiguous
    if (!at_once_) return at::empty_like(like_);
    return at::Tensor(at::detail::empty_strided_cuda(like_.sizes(), like_.strides(), like_.scalar_type(), like_.device()));
  }
  at::Tensor bytes(size_t n) const { return (*this)({(int64_t)n}, at::kByte); }

 private:
  const at::Tensor& like_;
  bool at_once_;
};

// Other threads run while memory is allocated and the kernels are launched: the allocator may wait for the GPU (when it gives
// cached blocks back) and a launch for room in the queue, and what they wait for may be up to another thread.
struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  NoGil() = default;
  NoGil(const NoGil&) = delete;
  ~NoGil() { PyEval_RestoreThread(state); }
};

// (O, LSE) or the library's status
PyObject* result(int rc, PyObject* out, const at::Tensor& o, PyObject* lse_arg, const at::Tensor& lse) {
  if (rc != 0) return PyLong_FromLong(rc);
  PyObject* a;
  PyObject* b;
  if (out != Py_None) { a = out; Py_INCREF(a); } else if ((a = THPVariable_Wrap(o)) == nullptr) return nullptr;
  if (lse_arg != Py_None || !lse.defined()) { b = lse_arg; Py_INCREF(b); }
  else if ((b = THPVariable_Wrap(lse)) == nullptr) { Py_DECREF(a); return nullptr; }
  PyObject* r = PyTuple_New(2);
  if (r == nullptr) { Py_DECREF(a); Py_DECREF(b); return nullptr; }
  PyTuple_SET_ITEM(r, 0, a);
  PyTuple_SET_ITEM(r, 1, b);
  return r;
}

// decode(shape, Q, kv, scale, n_splits, want_lse, out, lse, workspace, tail_k, tail_v, tail_len)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  hs_shape s;
  hs_kv kv;
  float scale;
  int32_t n_splits;
  if (n_args != 12 || !exact_tensor(a[1]) || !get_shape(a[0], &s) || !get_float(a[3], &scale) || !get_int(a[4], &n_splits) ||
      !PyBool_Check(a[5]))
    Py_RETURN_NONE;
  for (int i = 6; i < 11; i++)
    if (!none_or_tensor(a[i])) Py_RETURN_NONE;
  const at::Tensor& q = tensor(a[1]);
  if (!query_ok(q, s) || q.dim() < 2 || !get_kv(a[2], &kv)) Py_RETURN_NONE;
  const bool has_tail = a[11] != Py_None;
  int32_t tail_len = 0;
  const at::Tensor* rows = nullptr;
  if (has_tail) {
    for (int i = 9; i < 11; i++) {
      if (a[i] == Py_None) continue;
      const at::Tensor& t = tensor(a[i]);
      if (t.scalar_type() != q.scalar_type() || !t.is_contiguous() || t.dim() != 4 || t.size(0) != s.B || t.size(1) != s.Hkv ||
          t.size(2) != 64 || t.size(3) != s.D)
        Py_RETURN_NONE;
    }
    if (exact_tensor(a[11])) {
      rows = &tensor(a[11]);
      if (rows->scalar_type() != at::kInt || !rows->is_cuda() || rows->numel() != s.B || !rows->is_contiguous()) Py_RETURN_NONE;
    } else if (!get_int(a[11], &tail_len)) {
      Py_RETURN_NONE;
    }
  }
  const bool own_ws = a[8] == Py_None, own_o = a[6] == Py_None, own_lse = a[7] == Py_None && a[5] == Py_True;
  size_t need = 0;
  if (own_ws) {
    if (has_tail && n_splits == INT32_MAX) Py_RETURN_NONE;  // one more for the tail is no int32_t; the library refuses it
    const int n = has_tail ? (n_splits != 0 ? n_splits : g_hs.auto_splits(&s)) + 1 : n_splits;
    if (g_hs.workspace_bytes(&s, 2, n, &need) != 0) Py_RETURN_NONE;
  }
  void *ws_ptr = address(a[8]), *o_ptr = address(a[6]);
  float* lse_ptr = (float*)address(a[7]);
  const void *q_ptr = q.data_ptr(), *tk = address(a[9]), *tv = address(a[10]);
  const int32_t* lens = rows != nullptr ? (const int32_t*)rows->data_ptr() : nullptr;
  at::Tensor o, lse, ws;
  int rc;
  {
    NoGil others_run;
    if (own_ws || own_o || own_lse) {
      const NewTensors make(q);
      if (own_ws) { ws = make.bytes(need); ws_ptr = ws.data_ptr(); }
      if (own_o) { o = make.beside(); o_ptr = o.data_ptr(); }
      if (own_lse) { lse = make({q.size(0), q.size(1)}, at::kFloat); lse_ptr = (float*)lse.data_ptr(); }
    }
    void* st = current_stream();
    if (!has_tail) rc = g_hs.decode(&s, scale, n_splits, q_ptr, &kv, o_ptr, lse_ptr, ws_ptr, st);
    else if (rows != nullptr) rc = g_hs.decode_tail_rows(&s, scale, n_splits, q_ptr, &kv, tk, tv, lens, o_ptr, lse_ptr, ws_ptr, st);
    else rc = g_hs.decode_tail(&s, scale, n_splits, q_ptr, &kv, tk, tv, tail_len, o_ptr, lse_ptr, ws_ptr, st);
  }
  return result(rc, a[6], o, a[7], lse);
  END_HANDLE_TH_ERRORS
}

// decode_static(shape, Q, kv, scale, n_splits, out, lse)
PyObject* decode_static(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  hs_shape s;
  hs_kv kv;
  float scale;
  int32_t n_splits;
  if (n_args != 7 || !exact_tensor(a[1]) || !get_shape(a[0], &s) || !get_float(a[3], &scale) || !get_int(a[4], &n_splits) ||
      !exact_tensor(a[5]) || !none_or_tensor(a[6]))
    Py_RETURN_NONE;
  const at::Tensor& q = tensor(a[1]);
  if (!query_ok(q, s) || !get_kv(a[2], &kv)) Py_RETURN_NONE;
  const void* q_ptr = q.data_ptr();
  void *o_ptr = address(a[5]), *st = current_stream();
  float* lse_ptr = (float*)address(a[6]);
  int rc;
  {
    NoGil others_run;
    rc = g_hs.decode_static(&s, scale, n_splits, q_ptr, &kv, o_ptr, lse_ptr, st);
  }
  return result(rc, a[5], at::Tensor(), a[6], at::Tensor());
  END_HANDLE_TH_ERRORS
}

// prefill(shape, Q, kv, causal, scale, want_lse, out, lse, q_start, scratch): scratch None = not asked for yet; if the call wants
// any, (bytes, O, LSE) is returned with the outputs to hand in again: they come before the scratch, which the call can do
// without.  A tensor, or False for a call that runs without.
PyObject* prefill(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  hs_shape s;
  hs_kv kv;
  float scale;
  if (n_args != 10 || !exact_tensor(a[1]) || !get_shape(a[0], &s) || !PyBool_Check(a[3]) || !get_float(a[4], &scale) ||
      !PyBool_Check(a[5]) || !none_or_tensor(a[6]) || !none_or_tensor(a[7]) || !(a[9] == Py_False || none_or_tensor(a[9])))
    Py_RETURN_NONE;
  const at::Tensor& q = tensor(a[1]);
  if (!query_ok(q, s) || q.dim() != 4 || q.size(2) > INT32_MAX || !get_kv(a[2], &kv)) Py_RETURN_NONE;
  const int32_t Lq = (int32_t)q.size(2);
  int32_t at_pos = s.L - Lq;
  if (a[8] != Py_None && !get_int(a[8], &at_pos)) Py_RETURN_NONE;
  const int causal = a[3] == Py_True;
  size_t need = 0;
  void* ws_ptr = nullptr;
  if (a[9] == Py_None && g_hs.prefill_plan(&s, Lq, at_pos, causal, &kv, SIZE_MAX, nullptr, nullptr, &need) != 0) Py_RETURN_NONE;
  const bool own_o = a[6] == Py_None, own_lse = a[7] == Py_None && a[5] == Py_True, outputs_only = need != 0;
  if (exact_tensor(a[9])) {
    ws_ptr = address(a[9]);
    need = (size_t)tensor(a[9]).nbytes();
  }
  void* o_ptr = address(a[6]);
  float* lse_ptr = (float*)address(a[7]);
  const void* q_ptr = q.data_ptr();
  at::Tensor o, lse;
  int rc = 0;
  {
    NoGil others_run;
    if (own_o || own_lse) {
      const NewTensors make(q);
      if (own_o) { o = make.beside(); o_ptr = o.data_ptr(); }
      if (own_lse) { lse = make({q.size(0), q.size(1), q.size(2)}, at::kFloat); lse_ptr = (float*)lse.data_ptr(); }
    }
    if (!outputs_only)
      rc = g_hs.prefill(&s, Lq, at_pos, scale, causal, q_ptr, &kv, o_ptr, lse_ptr, ws_ptr, need, current_stream());
  }
  PyObject* r = result(rc, a[6], o, a[7], lse);
  if (!outputs_only || r == nullptr) return r;
  PyObject* first = Py_BuildValue("(nOO)", (Py_ssize_t)need, PyTuple_GET_ITEM(r, 0), PyTuple_GET_ITEM(r, 1));
  Py_DECREF(r);
  return first;
  END_HANDLE_TH_ERRORS
}

// append(shape, kv, tile, K, V, state_k, state_v, element_rule, overflow) -> status
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  hs_shape s;
  hs_kv kv;
  int32_t state_k, state_v, rule, tile = 0;
  if (n_args != 9 || !get_shape(a[0], &s) || !exact_tensor(a[3]) || !exact_tensor(a[4]) || !get_int(a[5], &state_k) ||
      !get_int(a[6], &state_v) || !get_int(a[7], &rule) || !none_or_tensor(a[8]))
    Py_RETURN_NONE;
  const at::Tensor &k = tensor(a[3]), &v = tensor(a[4]);
  if (k.scalar_type() != element_type(s) || v.scalar_type() != k.scalar_type() || k.dim() != 4 || k.strides() != v.strides() ||
      k.stride(3) != 1 || k.size(0) != s.B || k.size(1) != s.Hkv || k.size(3) != s.D || k.size(2) < 64 || k.size(2) % 64 != 0 ||
      k.size(2) / 64 > INT32_MAX || !get_kv(a[1], &kv))
    Py_RETURN_NONE;
  const int32_t n = (int32_t)(k.size(2) / 64);
  const at::Tensor* rows = nullptr;
  if (exact_tensor(a[2])) {
    rows = &tensor(a[2]);
    if (n != 1 || rows->scalar_type() != at::kInt || !rows->is_cuda() || rows->numel() != s.B || !rows->is_contiguous()) Py_RETURN_NONE;
  } else if (!get_int(a[2], &tile)) {
    Py_RETURN_NONE;
  }
  const int64_t strides[3] = {k.stride(0), k.stride(1), k.stride(2)};
  const void *kp = k.data_ptr(), *vp = v.data_ptr();
  const int32_t* at_rows = rows != nullptr ? (const int32_t*)rows->data_ptr() : nullptr;
  int32_t* over = (int32_t*)address(a[8]);
  void* st = current_stream();
  int rc;
  {
    NoGil others_run;
    rc = rows != nullptr ? g_hs.append_rows(&s, at_rows, state_k, state_v, rule, kp, vp, strides, &kv, over, st)
                         : g_hs.append(&s, tile, n, state_k, state_v, rule, kp, vp, strides, &kv, over, st);
  }
  return PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

// The eight buffers of a cache, in the order of kNames; an empty pool has none.
struct Pools {
  at::Tensor t[8];
  size_t bytes[8];
};

// They are made beside the tensor `like`, from the bytes that hs_kv_bytes has given (without the GIL); kv: the cache as the library sees it.
void make_pools(const hs_shape& s, const int32_t counts[5], const at::Tensor& like, int uniform, Pools* p, hs_kv* kv) {
  const NewTensors make(like);
  void** ptr[8] = {&kv->k_dense, &kv->k_nnz, &kv->k_meta, (void**)&kv->k_map, &kv->v_dense, &kv->v_nnz, &kv->v_meta, (void**)&kv->v_map};
  for (int i = 0; i < 8; i++) {
    const bool map = i == S_K_MAP || i == S_V_MAP;
    if (map || p->bytes[i] != 0)
      p->t[i] = map ? make({s.B, s.Hkv, s.L / 64}, at::kInt) : make.bytes(p->bytes[i]);
    *ptr[i] = p->t[i].defined() ? p->t[i].data_ptr() : nullptr;
  }
  kv->cap_dense_k = counts[1]; kv->cap_sparse_k = counts[2]; kv->cap_dense_v = counts[3]; kv->cap_sparse_v = counts[4];
  kv->uniform = uniform;
}

// The buffers as a tuple (None for an empty pool) with their bytes behind them.
PyObject* wrap_pools(const Pools& p) {
  PyObject* r = PyTuple_New(9);
  if (r == nullptr) return nullptr;
  size_t total = 0;
  for (int i = 0; i < 8; i++) {
    PyObject* t = Py_None;
    if (p.t[i].defined()) t = THPVariable_Wrap(p.t[i]);
    else Py_INCREF(t);
    if (t == nullptr) { Py_DECREF(r); return nullptr; }
    PyTuple_SET_ITEM(r, i, t);
    total += p.bytes[i];
  }
  PyObject* n = PyLong_FromSize_t(total);
  if (n == nullptr) { Py_DECREF(r); return nullptr; }
  PyTuple_SET_ITEM(r, 8, n);
  return r;
}

// slot == tile index: nothing skipped, one kind of tile per tensor
int counts_uniform(const int32_t c[5], int32_t T) {
  const int32_t k = c[1] > c[2] ? c[1] : c[2], v = c[3] > c[4] ? c[3] : c[4];
  return c[0] == 0 && (c[1] == 0 || c[2] == 0) && (c[3] == 0 || c[4] == 0) && k == T && v == T;
}

// pools(shape, counts, like): the buffers of a cache that the caller fills
PyObject* pools(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  hs_shape s;
  hs_kv kv;
  int32_t counts[5];
  Pools p;
  if (n_args != 3 || !get_shape(a[0], &s) || !get_counts(a[1], counts) || !exact_tensor(a[2]) || g_hs.kv_bytes(&s, counts, p.bytes) != 0)
    Py_RETURN_NONE;
  const at::Tensor& like = tensor(a[2]);
  {
    NoGil others_run;
    make_pools(s, counts, like, 0, &p, &kv);
  }
  return wrap_pools(p);
  END_HANDLE_TH_ERRORS
}

// (counts, pools, uniform) of a new cache, or the library's status
PyObject* new_cache(int rc, const int32_t c[5], const Pools& p, int uniform) {
  if (rc != 0) return PyLong_FromLong(rc);
  PyObject* bufs = wrap_pools(p);
  if (bufs == nullptr) return nullptr;
  return Py_BuildValue("([iiiii]Ni)", c[0], c[1], c[2], c[3], c[4], bufs, uniform);
}

// compress(shape, policy, K, V) -> (counts, pools, uniform); a policy of fractions, into a new cache
PyObject* compress(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  hs_shape s;
  hs_policy pol;
  hs_kv kv;
  if (n_args != 4 || !get_shape(a[0], &s) || !get_policy(a[1], &pol) || pol.state_k != nullptr || !exact_tensor(a[2]) || !exact_tensor(a[3]))
    Py_RETURN_NONE;
  const at::Tensor &k = tensor(a[2]), &v = tensor(a[3]);
  if (k.scalar_type() != element_type(s) || v.scalar_type() != k.scalar_type() || !k.is_cuda() || !v.is_cuda() || k.dim() != 4 ||
      k.stride(3) != 1 || k.strides() != v.strides())
    Py_RETURN_NONE;
  int32_t counts[5];
  size_t need = 0;
  Pools p;
  if (g_hs.tile_counts(&s, &pol, counts) != 0 || g_hs.workspace_bytes(&s, 0, 0, &need) != 0 || g_hs.kv_bytes(&s, counts, p.bytes) != 0)
    Py_RETURN_NONE;
  const int uniform = counts_uniform(counts, s.L / 64);
  const int64_t strides[3] = {k.stride(0), k.stride(1), k.stride(2)};
  const void *kp = k.data_ptr(), *vp = v.data_ptr();
  int rc;
  {
    NoGil others_run;
    make_pools(s, counts, k, uniform, &p, &kv);
    const at::Tensor ws = NewTensors(k).bytes(need < 16 ? 16 : need);
    rc = g_hs.compress(&s, &pol, kp, vp, strides, &kv, ws.data_ptr(), current_stream());
  }
  return new_cache(rc, counts, p, uniform);
  END_HANDLE_TH_ERRORS
}

// recompress(shape, cache, target, counts, overflow) -> (counts, pools, uniform); a target of whole fractions, into a new cache
PyObject* recompress(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  hs_shape s;
  hs_policy pol;
  hs_kv src, dst;
  int32_t c[5];
  Pools p;
  if (n_args != 5 || !get_shape(a[0], &s) || !get_kv(a[1], &src) || !get_policy(a[2], &pol) || pol.state_k != nullptr ||
      pol.tile_scores != nullptr || !get_counts(a[3], c) || !none_or_tensor(a[4]) || g_hs.kv_bytes(&s, c, p.bytes) != 0)
    Py_RETURN_NONE;
  PyObject* map = PyObject_GetAttr(a[1], g_names[S_K_MAP]);
  if (map == nullptr) return nullptr;
  if (!exact_tensor(map)) { Py_DECREF(map); Py_RETURN_NONE; }
  const at::Tensor like = tensor(map);
  Py_DECREF(map);
  const int32_t T = s.L / 64, k = c[1] > c[2] ? c[1] : c[2], v = c[3] > c[4] ? c[3] : c[4];
  const bool whole = pol.skip_frac == 0.0 && (pol.sparse_frac_k == 0.0 || pol.sparse_frac_k == 1.0) &&
                     (pol.sparse_frac_v == 0.0 || pol.sparse_frac_v == 1.0);
  // slot == tile survives when nothing was skipped before and each tensor ends up in one kind
  const int uniform = src.uniform != 0 && whole && (c[1] == 0 || c[2] == 0) && (c[3] == 0 || c[4] == 0) && k == T && v == T;
  int32_t* over = (int32_t*)address(a[4]);
  int rc;
  {
    NoGil others_run;
    make_pools(s, c, like, uniform, &p, &dst);
    rc = g_hs.recompress(&s, &pol, &src, &dst, nullptr, over, current_stream());
  }
  return new_cache(rc, c, p, uniform);
  END_HANDLE_TH_ERRORS
}

// bind(addresses in the order of Entries, HsShape, HsPolicy, PackedKV)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  constexpr Py_ssize_t n = sizeof(Entries) / sizeof(void*);
  if (n_args != 4 || !PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != n || !PyType_Check(a[1]) || !PyType_Check(a[2]) || !PyType_Check(a[3])) {
    PyErr_SetString(PyExc_TypeError, "bind(addresses, shape type, policy type, cache type)");
    return nullptr;
  }
  void* p[n];
  for (Py_ssize_t i = 0; i < n; i++) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[0], i));
    if (p[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry");
      return nullptr;
    }
  }
  memcpy(&g_hs, p, sizeof(p));
  PyTypeObject** types[3] = {&g_shape_type, &g_policy_type, &g_kv_type};
  for (int i = 0; i < 3; i++) {
    Py_INCREF(a[1 + i]);
    Py_XDECREF(*types[i]);
    *types[i] = (PyTypeObject*)a[1 + i];
  }
  Py_RETURN_NONE;
}

#define HS_FN(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {HS_FN(bind), HS_FN(decode), HS_FN(decode_static), HS_FN(prefill), HS_FN(append), HS_FN(pools), HS_FN(compress), HS_FN(recompress),
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_hs_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#define HS_STR_(x) #x
#define HS_STR(x) HS_STR_(x)

PyMODINIT_FUNC PyInit__hs_torch() {
  for (int i = 0; i < N_NAMES; i++) {
    g_names[i] = PyUnicode_InternFromString(kNames[i]);
    if (g_names[i] == nullptr) return nullptr;
  }
  PyObject* m = PyModule_Create(&kModule);
  // what the binding compares before it uses the module
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", "torch " HS_TORCH_VERSION ", Python " HS_STR(PY_MAJOR_VERSION) "." HS_STR(PY_MINOR_VERSION)) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
