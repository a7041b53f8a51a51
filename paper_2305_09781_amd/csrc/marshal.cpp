// Argument marshalling of the Python binding: tensors to pointers, strides and sizes, the layout checks of binding.py, outputs
// and workspaces where the caller brings none, and the call into libspectree. Host code only.
//
// Why it is native: a small layer is 7 to 12 us on the device, and the same work in Python (shape and stride tuples, a ctypes
// object per pointer, two foreign calls, a stream object) took 17 to 25 us a call, so that the device waited for the caller.
// Measured, us a pass among others: a float32 layer of one request 16.7 -> 10.6, a paged layer of 5 x 12 heads 20.7 -> 11.0,
// greedy verification of 4 x 110 x 1051 bfloat16 logits 11.9 -> 8.5, eight tree levels and a merge 88.4 -> 58.6.
//
// Every function takes its arguments by position, as binding.py passes them, None where an optional one is absent. The GIL is
// released around the library's calls, as ctypes does, and around allocations, as torch does.
#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <vector>

#include "spec_tree.h"

namespace {

using at::Tensor;

PyObject* g_spec_error = nullptr;       // binding.SpecError(code, where)
PyObject* g_argument_error = nullptr;   // what ctypes raises for an argument of another type
PyObject* g_stream = nullptr;           // binding._stream(stream): the handle, of the current stream for None

[[noreturn]] void fail(PyObject* type, const std::string& what) {
  PyErr_SetString(type, what.c_str());
  throw python_error();
}
[[noreturn]] void value_error(const std::string& what) { fail(PyExc_ValueError, what); }

void check(int rc, const char* where) {
  if (rc == SPEC_OK) return;
  PyObject* e = PyObject_CallFunction(g_spec_error, "is", rc, where);
  if (e != nullptr) {
    PyErr_SetObject(g_spec_error, e);
    Py_DECREF(e);
  }
  throw python_error();
}

struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};
template <class Call>
void call(const char* where, Call&& f) {
  int rc;
  {
    NoGil released;
    rc = f();
  }
  check(rc, where);
}

// One call's arguments, read in order.
struct Args {
  PyObject* const* at;
  Py_ssize_t left;
  PyObject* next() {
    if (left <= 0) fail(PyExc_TypeError, "too few arguments");
    --left;
    return *at++;
  }
  const Tensor* tensor_or_none() {
    PyObject* o = next();
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, std::string("expected a tensor, got ") + Py_TYPE(o)->tp_name);
    return &THPVariable_Unpack(o);
  }
  const Tensor& tensor() {
    const Tensor* t = tensor_or_none();
    if (t == nullptr) fail(PyExc_TypeError, "expected a tensor, got None");
    return *t;
  }
  void* address() {
    void* p = PyLong_AsVoidPtr(next());
    if (p == nullptr && PyErr_Occurred()) throw python_error();
    return p;
  }
  int32_t i32() {   // an int and nothing else, in 32 bits, as ctypes takes it
    PyObject* o = next();
    if (!PyLong_Check(o)) fail(g_argument_error, std::string("int expected instead of ") + Py_TYPE(o)->tp_name + " instance");
    return (int32_t)PyLong_AsUnsignedLongMask(o);
  }
  int32_t to_i32() { return as_i32(next()); }   // int(argument)
  static int32_t as_i32(PyObject* o) {
    if (PyLong_CheckExact(o)) return (int32_t)PyLong_AsUnsignedLongMask(o);
    PyObject* n = PyNumber_Long(o);
    if (n == nullptr) throw python_error();
    const int32_t v = (int32_t)PyLong_AsUnsignedLongMask(n);
    Py_DECREF(n);
    return v;
  }
  double to_double() {   // float(argument)
    PyObject* o = next();
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    PyObject* n = PyNumber_Float(o);
    if (n == nullptr) throw python_error();
    const double v = PyFloat_AS_DOUBLE(n);
    Py_DECREF(n);
    return v;
  }
};

void* handle(PyObject* stream) {
  PyObject* h = PyObject_CallFunctionObjArgs(g_stream, stream, nullptr);
  if (h == nullptr) throw python_error();
  void* p = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  if (p == nullptr && PyErr_Occurred()) throw python_error();
  return p;
}

void* ptr(const Tensor& t) { return t.data_ptr(); }
void* ptr(const Tensor* t) { return t == nullptr ? nullptr : t->data_ptr(); }
template <class T, class X>
T* as(X&& t) { return (T*)ptr(t); }

void same_layout(const Tensor& a, const Tensor& b, const char* what) {
  if (a.sizes() != b.sizes() || a.strides() != b.strides() || a.scalar_type() != b.scalar_type())
    value_error(std::string(what) + " must share shape, strides and dtype");
}
void need_dims(const Tensor& t, int64_t dims, const char* what) {
  if (t.dim() != dims) value_error(std::string(what) + " must have " + std::to_string(dims) + " dimensions");
}
int32_t dtype_code(const Tensor& t) {
  if (t.scalar_type() == at::kFloat) return SPEC_F32;
  if (t.scalar_type() == at::kBFloat16) return SPEC_BF16;
  fail(PyExc_TypeError, std::string("unsupported dtype ") + c10::toString(t.scalar_type()));
}
// (an allocation may wait for the device: other threads run meanwhile, as they do under torch.empty)
Tensor empty(at::IntArrayRef shape, at::ScalarType type, const Tensor& like) {
  NoGil released;
  return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}
Tensor empty_as(const Tensor& like) {
  NoGil released;
  return at::empty_like(like);
}
PyObject* wrap(const Tensor& t) {
  PyObject* o = THPVariable_Wrap(t);
  if (o == nullptr) throw python_error();
  return o;
}
template <size_t N>
PyObject* wrap(const Tensor (&ts)[N]) {
  PyObject* r = PyTuple_New(N);
  if (r == nullptr) throw python_error();
  for (size_t i = 0; i < N; ++i) PyTuple_SET_ITEM(r, i, wrap(ts[i]));
  return r;
}

// ------------------------------------------------------------------------------------------------
// descriptors
// ------------------------------------------------------------------------------------------------
struct Plan {
  int32_t chunk_keys = 0, balanced_wgs = 0, heads_per_wg = 0;
  explicit Plan(PyObject* o) {
    int32_t* to[3] = {&chunk_keys, &balanced_wgs, &heads_per_wg};
    for (int i = 0; i < 3; ++i) {   // int(plan[i]), of a tuple or of anything that has items 0 to 2
      PyObject* at = PyTuple_CheckExact(o) ? nullptr : PyLong_FromLong(i);
      PyObject* v = at == nullptr ? PySequence_GetItem(o, i) : PyObject_GetItem(o, at);
      Py_XDECREF(at);
      if (v == nullptr) throw python_error();
      struct Release { PyObject* o; ~Release() { Py_DECREF(o); } } release{v};
      *to[i] = Args::as_i32(v);
    }
  }
};

void fill_desc(spec_attn_desc_t* d, const Tensor& q, const Tensor& cache, int32_t max_prefix_len, double softmax_scale,
               const Tensor* k_new, const Plan& plan, const Tensor* block_table) {
  need_dims(q, 4, "q");
  need_dims(cache, 4, block_table ? "pool" : "cache");
  const int64_t B = q.size(0), N = q.size(1), H = q.size(2), D = q.size(3), H_kv = cache.size(1);
  if (block_table != nullptr) {
    if (cache.size(3) != D || q.stride(3) != 1 || cache.stride(3) != 1)
      value_error("q must be [B,N,H,D], pool [n_blocks,H_kv,block_tokens,D], D contiguous");
    if (block_table->scalar_type() != at::kInt || block_table->dim() != 2 || block_table->size(0) != B || !block_table->is_contiguous())
      value_error("block_table must be contiguous int32 [B, max_blocks]");
  } else if (cache.size(0) != B || cache.size(3) != D || q.stride(3) != 1 || cache.stride(3) != 1) {
    value_error("q must be [B,N,H,D], cache [B,H_kv,S_cap,D], D contiguous");
  }
  int64_t ns[3] = {0, 0, 0};
  if (k_new != nullptr) {
    if (k_new->dim() != 4 || k_new->size(0) != B || k_new->size(1) != N || k_new->size(2) != H_kv || k_new->size(3) != D ||
        k_new->stride(3) != 1)
      value_error("k_new / v_new must be [B,N,H_kv,D], D contiguous");
    for (int i = 0; i < 3; ++i) ns[i] = k_new->stride(i);
  }
  d->B = (int32_t)B; d->H = (int32_t)H; d->H_kv = (int32_t)H_kv; d->D = (int32_t)D; d->N = (int32_t)N;
  d->S_cap = (int32_t)(block_table != nullptr ? block_table->size(1) * cache.size(2) : cache.size(2));
  d->dtype = dtype_code(q);
  d->max_prefix_len = max_prefix_len;
  d->q_stride_b = q.stride(0); d->q_stride_n = q.stride(1); d->q_stride_h = q.stride(2);
  d->kv_stride_b = cache.stride(0); d->kv_stride_h = cache.stride(1); d->kv_stride_s = cache.stride(2);
  d->new_stride_b = ns[0]; d->new_stride_n = ns[1]; d->new_stride_h = ns[2];
  d->softmax_scale = (float)softmax_scale;
  d->plan_chunk_keys = plan.chunk_keys; d->plan_balanced_wgs = plan.balanced_wgs; d->plan_heads_per_wg = plan.heads_per_wg;
}
spec_kv_pages_t make_pages(const Tensor& pool, const Tensor& block_table) {
  spec_kv_pages_t p = {};
  p.block_table = as<int32_t>(block_table);
  p.max_blocks = (int32_t)block_table.size(1);
  p.block_tokens = (int32_t)pool.size(2);
  p.n_blocks = (int32_t)pool.size(0);
  return p;
}

// fill_desc(desc address, pages address or 0, q, cache or pool, block_table, max_prefix_len, softmax_scale, k_new, plan)
PyObject* py_fill_desc(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  auto* d = (spec_attn_desc_t*)a.address();
  auto* pages = (spec_kv_pages_t*)a.address();
  const Tensor &q = a.tensor(), &cache = a.tensor();
  const Tensor* table = a.tensor_or_none();
  const int32_t max_prefix_len = a.to_i32();
  const double scale = a.to_double();
  const Tensor* k_new = a.tensor_or_none();
  fill_desc(d, q, cache, max_prefix_len, scale, k_new, Plan(a.next()), table);
  if (table != nullptr) *pages = make_pages(cache, *table);
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

// ------------------------------------------------------------------------------------------------
// attention: all entry points that attend. flags, of what the entry point is: 1 paged (and says so), 2 on the library's own
// scratch, 4 with the rotary embedding, 8 with the append
// (q, k_new, v_new, k_cache, v_cache, block_table, parent, depth, prefix_len, cos, sin, out, workspace, status, max_prefix_len,
//  softmax_scale, stream, desc address or 0, plan, flags) -> out
// ------------------------------------------------------------------------------------------------
PyObject* py_tree_attention(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor& q = a.tensor();
  const Tensor *k_new = a.tensor_or_none(), *v_new = a.tensor_or_none();
  const Tensor &kc = a.tensor(), &vc = a.tensor();
  const Tensor* table = a.tensor_or_none();
  const Tensor &parent = a.tensor(), &depth = a.tensor(), &prefix_len = a.tensor();
  const Tensor *cos = a.tensor_or_none(), *sin = a.tensor_or_none(), *out_given = a.tensor_or_none();
  const Tensor *ws_given = a.tensor_or_none(), *status = a.tensor_or_none();
  PyObject* max_prefix_obj = a.next();
  PyObject* scale_obj = a.next();
  PyObject* on_stream = a.next();
  const auto* desc = (const spec_attn_desc_t*)a.address();
  PyObject* plan = a.next();
  const int32_t flags = a.i32();
  const bool pools = flags & 1, own_scratch = flags & 2;
  if ((pools && table == nullptr) || ((flags & 4) && (cos == nullptr || sin == nullptr)) || ((flags & 8) && (k_new == nullptr || v_new == nullptr)) ||
      (own_scratch && out_given == nullptr))
    fail(PyExc_TypeError, "a tensor this entry point needs is None");

  same_layout(kc, vc, pools ? "k_pool and v_pool" : "k_cache and v_cache");
  if (k_new != nullptr && v_new != nullptr && !pools) same_layout(*k_new, *v_new, "k_new and v_new");
  for (const Tensor* tab : {cos, sin})
    if (tab != nullptr && (tab->scalar_type() != at::kFloat || tab->dim() != 2 || tab->size(1) != k_new->size(-1) / 2 || !tab->is_contiguous()))
      value_error("rope tables must be contiguous float32 [rope_len, D/2]");
  const Tensor out = out_given != nullptr ? *out_given : empty_as(q);
  same_layout(q, out, "q and out");
  spec_attn_desc_t d;
  spec_kv_pages_t pages;
  if (desc != nullptr) {
    d = *desc;
  } else {
    Args rest{&scale_obj, 1};
    const int32_t max_prefix_len = Args::as_i32(max_prefix_obj);
    fill_desc(&d, q, kc, max_prefix_len, rest.to_double(), k_new, Plan(plan), table);
  }
  if (table != nullptr) pages = make_pages(kc, *table);
  Tensor ws;
  size_t ws_bytes = 0;
  if (!own_scratch) {
    if (ws_given != nullptr) {
      ws = *ws_given;
    } else {
      const size_t need = table != nullptr ? spec_tree_attention_paged_workspace_bytes(&d, &pages) : spec_tree_attention_workspace_bytes(&d);
      if (need > 0) ws = empty({(int64_t)need}, at::kByte, q);
    }
    if (ws.defined()) ws_bytes = (size_t)ws.numel() * ws.element_size();
  }
  if (pools && k_new != nullptr && v_new != nullptr) same_layout(*k_new, *v_new, "k_new and v_new");
  const auto *par = as<int32_t>(parent), *dep = as<int32_t>(depth), *pl = as<int32_t>(prefix_len);
  const auto *cs = as<float>(cos), *sn = as<float>(sin);
  void *qp = ptr(q), *kn = ptr(k_new), *vn = ptr(v_new), *kp = ptr(kc), *vp = ptr(vc), *op = ptr(out), *wp = ws.defined() ? ptr(ws) : nullptr;
  auto* st = as<int32_t>(status);
  const int32_t rope_len = cos != nullptr ? (int32_t)cos->size(0) : 0;
  void* stream = handle(on_stream);
  if (own_scratch) {
    call("spec_tree_attention_append_static", [&] { return spec_tree_attention_append_static(&d, qp, kn, vn, kp, vp, par, dep, pl, op, st, stream); });
  } else if (cos != nullptr && table != nullptr) {
    call("spec_tree_attention_append_rope_paged", [&] {
      return spec_tree_attention_append_rope_paged(&d, &pages, qp, kn, vn, kp, vp, par, dep, pl, cs, sn, rope_len, op, wp, ws_bytes, st, stream); });
  } else if (cos != nullptr) {
    call("spec_tree_attention_append_rope", [&] {
      return spec_tree_attention_append_rope(&d, qp, kn, vn, kp, vp, par, dep, pl, cs, sn, rope_len, op, wp, ws_bytes, st, stream); });
  } else if (table != nullptr && k_new != nullptr) {
    call("spec_tree_attention_append_paged", [&] {
      return spec_tree_attention_append_paged(&d, &pages, qp, kn, vn, kp, vp, par, dep, pl, op, wp, ws_bytes, st, stream); });
  } else if (table != nullptr) {
    call("spec_tree_attention_paged", [&] { return spec_tree_attention_paged(&d, &pages, qp, kp, vp, par, dep, pl, op, wp, ws_bytes, st, stream); });
  } else if (k_new != nullptr) {
    call("spec_tree_attention_append", [&] {
      return spec_tree_attention_append(&d, qp, kn, vn, kp, vp, par, dep, pl, op, wp, ws_bytes, st, stream); });
  } else {
    call("spec_tree_attention", [&] { return spec_tree_attention(&d, qp, kp, vp, par, dep, pl, op, wp, ws_bytes, st, stream); });
  }
  return wrap(out);
  END_HANDLE_TH_ERRORS
}

// ------------------------------------------------------------------------------------------------
// verification
// ------------------------------------------------------------------------------------------------
// Outputs: whether the caller brings them, then the tensors themselves (None among those passes a null pointer).
template <int N>
struct Given {
  bool any;
  Tensor at[N];
  explicit Given(Args& a) {
    const int brought = PyObject_IsTrue(a.next());
    if (brought < 0) throw python_error();
    any = brought;
    for (Tensor& t : at) {
      const Tensor* g = a.tensor_or_none();
      if (g != nullptr) t = *g;
    }
  }
  int32_t* i32(int i) const { return at[i].defined() ? as<int32_t>(at[i]) : nullptr; }
};
int32_t steps(PyObject* lmax, int64_t N) {   // Lmax (None: N)
  if (lmax == Py_None) return (int32_t)N;
  Args one{&lmax, 1};
  return one.i32();
}
// path, len and tokens of a walk, and (outputs of four) the nodes' arg-max, where the caller brings none
template <int COUNT>
void make_walk(Given<COUNT>& o, int64_t B, int64_t N, int32_t Lmax, const Tensor& like) {
  if (o.any) return;
  o.at[0] = empty({B, Lmax}, at::kInt, like);
  o.at[1] = empty({B}, at::kInt, like);
  o.at[2] = empty({B, Lmax}, at::kInt, like);
  if (COUNT > 3) o.at[COUNT - 1] = empty({B, N}, at::kInt, like);
}

// (logits, tree_token, tree_parent, Lmax, status, stream, brought, path, len, tokens, argmax) -> the last four
PyObject* py_verify_greedy(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor &logits = a.tensor(), &token = a.tensor(), &parent = a.tensor();
  PyObject* lmax = a.next();
  const Tensor* status = a.tensor_or_none();
  PyObject* on_stream = a.next();
  Given<4> o(a);
  need_dims(logits, 3, "logits");
  const int64_t B = logits.size(0), N = logits.size(1), V = logits.size(2);
  const int32_t Lmax = steps(lmax, N);
  make_walk(o, B, N, Lmax, logits);
  const int32_t dtype = dtype_code(logits);
  const void* lg = ptr(logits);
  const auto *tk = as<int32_t>(token), *pr = as<int32_t>(parent);
  int32_t *pp = o.i32(0), *lp = o.i32(1), *tp = o.i32(2), *ap = o.i32(3), *st = as<int32_t>(status);
  void* stream = handle(on_stream);
  call("spec_verify_greedy", [&] {
    return spec_verify_greedy((int32_t)B, (int32_t)N, (int32_t)V, dtype, lg, tk, pr, Lmax, pp, lp, tp, ap, nullptr, 0, st, stream); });
  return wrap(o.at);
  END_HANDLE_TH_ERRORS
}

// (logits, from statistics, node_max, node_sumexp, probs_ssm, ssm_row, tree_token, tree_parent, u_accept, u_order, u_final,
//  temperature, Lmax, workspace, status, stream, brought, path, len, tokens) -> the last three
PyObject* py_verify_stochastic(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor& logits = a.tensor();
  const bool stats = a.next() == Py_True;
  const Tensor *mx = a.tensor_or_none(), *se = a.tensor_or_none();
  const Tensor &probs = a.tensor(), &row = a.tensor(), &token = a.tensor(), &parent = a.tensor();
  const Tensor &ua = a.tensor(), &uo = a.tensor(), &uf = a.tensor();
  const double temperature = a.to_double();
  PyObject* lmax = a.next();
  const Tensor *ws_given = a.tensor_or_none(), *status = a.tensor_or_none();
  PyObject* on_stream = a.next();
  Given<3> o(a);
  need_dims(logits, 3, "logits");
  const int64_t B = logits.size(0), N = logits.size(1), V = logits.size(2);
  if (probs.scalar_type() != at::kFloat || (probs.numel() != 0 && (probs.dim() < 2 || probs.size(1) != V)) || !probs.is_contiguous())
    value_error("probs_ssm must be contiguous float32 [R,V]");
  if (stats)
    for (const Tensor* t : {mx, se})
      if (t == nullptr || t->scalar_type() != at::kFloat || t->numel() != B * N || !t->is_contiguous())
        value_error("node_max / node_sumexp must be contiguous float32 with B*N entries");
  Tensor ws;
  if (ws_given != nullptr) {
    ws = *ws_given;
  } else {
    const size_t need = stats ? spec_verify_stochastic_stats_workspace_bytes((int32_t)B, (int32_t)V)
                              : spec_verify_stochastic_workspace_bytes((int32_t)B, (int32_t)N, (int32_t)V);
    ws = empty({(int64_t)need}, at::kByte, logits);
  }
  const int32_t Lmax = steps(lmax, N);
  make_walk(o, B, N, Lmax, logits);
  const size_t ws_bytes = stats ? (size_t)ws.numel() : (size_t)ws.numel() * ws.element_size();
  const int32_t dtype = dtype_code(logits), R = (int32_t)probs.size(0);
  const void* lg = ptr(logits);
  const auto *mp = as<float>(mx), *sp = as<float>(se), *pb = as<float>(probs), *uap = as<float>(ua), *uop = as<float>(uo), *ufp = as<float>(uf);
  const auto *rw = as<int32_t>(row), *tk = as<int32_t>(token), *pr = as<int32_t>(parent);
  int32_t *pp = o.i32(0), *lp = o.i32(1), *tp = o.i32(2), *st = as<int32_t>(status);
  void* wp = ptr(ws);
  const float temp = (float)temperature;
  void* stream = handle(on_stream);
  if (stats)
    call("spec_verify_stochastic_stats", [&] {
      return spec_verify_stochastic_stats((int32_t)B, (int32_t)N, (int32_t)V, dtype, lg, mp, sp, pb, R, rw, tk, pr, uap, uop, ufp, temp, Lmax,
                                          pp, lp, tp, wp, ws_bytes, st, stream); });
  else
    call("spec_verify_stochastic", [&] {
      return spec_verify_stochastic((int32_t)B, (int32_t)N, (int32_t)V, dtype, lg, pb, R, rw, tk, pr, uap, uop, ufp, temp, Lmax, pp, lp, tp,
                                    wp, ws_bytes, st, stream); });
  return wrap(o.at);
  END_HANDLE_TH_ERRORS
}

// ------------------------------------------------------------------------------------------------
// token trees
// ------------------------------------------------------------------------------------------------
// (ssm_logits, k, child_slot, tree_token, status, stream)
PyObject* py_expand_topk(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor& logits = a.tensor();
  const int32_t k = a.i32();
  const Tensor &slot = a.tensor(), &tree = a.tensor();
  const Tensor* status = a.tensor_or_none();
  PyObject* on_stream = a.next();
  need_dims(logits, 3, "ssm_logits");
  const int64_t B = logits.size(0), F = logits.size(1), V = logits.size(2), N = tree.size(1);
  if (slot.scalar_type() != at::kInt || slot.dim() != 2 || slot.size(0) != F || slot.size(1) != k || !slot.is_contiguous())
    value_error("child_slot must be contiguous int32 [F, k]");
  if (!logits.is_contiguous() || !tree.is_contiguous() || tree.scalar_type() != at::kInt)
    value_error("ssm_logits and tree_token (int32) must be contiguous");
  const int32_t dtype = dtype_code(logits);
  const void* lg = ptr(logits);
  const auto* sl = as<int32_t>(slot);
  int32_t *tr = as<int32_t>(tree), *st = as<int32_t>(status);
  void* stream = handle(on_stream);
  call("spec_tree_expand_topk", [&] {
    return spec_tree_expand_topk((int32_t)B, (int32_t)F, (int32_t)V, dtype, lg, k, sl, (int32_t)N, tr, st, stream); });
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

// (in_parent, in_token, in_size, Nout, status, stream, want_node_map) -> parent, depth, token, ssm, size, node_map or None
PyObject* py_tree_merge(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor &par = a.tensor(), &tok = a.tensor(), &size = a.tensor();
  const int32_t Nout = a.i32();
  const Tensor* status = a.tensor_or_none();
  PyObject* on_stream = a.next();
  const int want_map = PyObject_IsTrue(a.next());
  if (want_map < 0) throw python_error();
  need_dims(par, 3, "in_parent");
  const int64_t B = par.size(0), M = par.size(1), Nin = par.size(2);
  for (const Tensor* t : {&par, &tok, &size})
    if (t->scalar_type() != at::kInt || !t->is_contiguous()) value_error("tree_merge inputs must be contiguous int32");
  Tensor o[6];
  for (int i = 0; i < 4; ++i) o[i] = empty({B, Nout}, at::kInt, par);
  o[4] = empty({B}, at::kInt, par);
  if (want_map) o[5] = empty({B, M, Nin}, at::kInt, par);
  const auto *pp = as<int32_t>(par), *tp = as<int32_t>(tok), *sp = as<int32_t>(size);
  int32_t* op[6];
  for (int i = 0; i < 6; ++i) op[i] = o[i].defined() ? as<int32_t>(o[i]) : nullptr;
  int32_t* st = as<int32_t>(status);
  void* stream = handle(on_stream);
  call("spec_tree_merge", [&] {
    return spec_tree_merge((int32_t)B, (int32_t)M, (int32_t)Nin, pp, tp, sp, Nout, op[0], op[1], op[2], op[3], op[4], op[5], st, stream); });
  return wrap(o);   // (an undefined tensor is None)
  END_HANDLE_TH_ERRORS
}

// ------------------------------------------------------------------------------------------------
// LM head
// ------------------------------------------------------------------------------------------------
struct Head {
  const Tensor &hidden, &weight;
  int64_t M, K, V;
  Head(const Tensor& h, const Tensor& w) : hidden(h), weight(w) {
    if (h.scalar_type() != at::kBFloat16 || w.scalar_type() != at::kBFloat16 || h.dim() != 2 || w.dim() != 2 || h.size(1) != w.size(1) ||
        !h.is_contiguous() || !w.is_contiguous())
      value_error("hidden [M,K] and weight [V,K] must be contiguous bf16 with the same K");
    M = h.size(0); K = h.size(1); V = w.size(0);
  }
  Tensor workspace(const Tensor* given, size_t need) const {
    return given != nullptr ? *given : empty({(int64_t)std::max<size_t>(need, 256)}, at::kByte, hidden);
  }
};

// (hidden, weight, want_max, workspace, stream) -> node_argmax, node_max or None
PyObject* py_lm_head_argmax(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor &hidden = a.tensor(), &weight = a.tensor();
  const int want_max = PyObject_IsTrue(a.next());
  if (want_max < 0) throw python_error();
  const Tensor* ws_given = a.tensor_or_none();
  PyObject* on_stream = a.next();
  const Head h(hidden, weight);
  Tensor o[2];
  o[0] = empty({h.M}, at::kInt, hidden);
  if (want_max) o[1] = empty({h.M}, at::kFloat, hidden);
  const Tensor ws = h.workspace(ws_given, spec_lm_head_argmax_workspace_bytes((int32_t)h.M, (int32_t)h.V));
  const void *hp = ptr(hidden), *wt = ptr(weight);
  int32_t* ap = as<int32_t>(o[0]);
  float* mp = want_max ? as<float>(o[1]) : nullptr;
  void* wp = ptr(ws);
  const size_t ws_bytes = (size_t)ws.numel();
  void* stream = handle(on_stream);
  call("spec_lm_head_argmax", [&] { return spec_lm_head_argmax((int32_t)h.M, (int32_t)h.K, (int32_t)h.V, hp, wt, ap, mp, wp, ws_bytes, stream); });
  return wrap(o);
  END_HANDLE_TH_ERRORS
}

// (hidden, weight, tree_token, tree_parent, Lmax, workspace, status, stream, brought, path, len, tokens, argmax) -> the last four
PyObject* py_verify_greedy_lm_head(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor &hidden = a.tensor(), &weight = a.tensor(), &token = a.tensor(), &parent = a.tensor();
  PyObject* lmax = a.next();
  const Tensor *ws_given = a.tensor_or_none(), *status = a.tensor_or_none();
  PyObject* on_stream = a.next();
  Given<4> o(a);
  const Head h(hidden, weight);
  need_dims(token, 2, "tree_token");
  const int64_t B = token.size(0), N = token.size(1);
  if (h.M != B * N) value_error("hidden must have B*N rows");
  const int32_t Lmax = steps(lmax, N);
  make_walk(o, B, N, Lmax, hidden);
  const Tensor ws = h.workspace(ws_given, spec_lm_head_argmax_workspace_bytes((int32_t)h.M, (int32_t)h.V));
  const void *hp = ptr(hidden), *wt = ptr(weight);
  const auto *tk = as<int32_t>(token), *pr = as<int32_t>(parent);
  int32_t *pp = o.i32(0), *lp = o.i32(1), *tp = o.i32(2), *ap = o.i32(3), *st = as<int32_t>(status);
  void* wp = ptr(ws);
  const size_t ws_bytes = (size_t)ws.numel();
  void* stream = handle(on_stream);
  call("spec_verify_greedy_lm_head", [&] {
    return spec_verify_greedy_lm_head((int32_t)B, (int32_t)N, (int32_t)h.K, (int32_t)h.V, hp, wt, tk, pr, Lmax, pp, lp, tp, ap, wp, ws_bytes, st,
                                      stream); });
  return wrap(o.at);
  END_HANDLE_TH_ERRORS
}

// (hidden, weight, temperature, workspace, stream, brought, logits, argmax, max, sumexp) -> the last four
PyObject* py_lm_head_logits_stats(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  const Tensor &hidden = a.tensor(), &weight = a.tensor();
  const double temperature = a.to_double();
  const Tensor* ws_given = a.tensor_or_none();
  PyObject* on_stream = a.next();
  Given<4> o(a);
  const Head h(hidden, weight);
  if (!o.any) {
    o.at[0] = empty({h.M, h.V}, at::kBFloat16, hidden);
    o.at[1] = empty({h.M}, at::kInt, hidden);
    o.at[2] = empty({h.M}, at::kFloat, hidden);
    o.at[3] = empty({h.M}, at::kFloat, hidden);
  }
  const Tensor ws = h.workspace(ws_given, spec_lm_head_logits_stats_workspace_bytes((int32_t)h.M, (int32_t)h.V));
  const void *hp = ptr(hidden), *wt = ptr(weight);
  void* op[4];
  for (int i = 0; i < 4; ++i) op[i] = o.i32(i);
  void* wp = ptr(ws);
  const size_t ws_bytes = (size_t)ws.numel();
  const float temp = (float)temperature;
  void* stream = handle(on_stream);
  call("spec_lm_head_logits_stats", [&] {
    return spec_lm_head_logits_stats((int32_t)h.M, (int32_t)h.K, (int32_t)h.V, hp, wt, temp, op[0], (int32_t*)op[1], (float*)op[2],
                                     (float*)op[3], wp, ws_bytes, stream); });
  return wrap(o.at);
  END_HANDLE_TH_ERRORS
}

// ------------------------------------------------------------------------------------------------
// commit: (k_caches, v_caches, block_table, path, len, prefix_len, N, prefix_len_out, status, stream) -> prefix_len_out
// ------------------------------------------------------------------------------------------------
struct Caches {   // a sequence of caches, held while its pointers are in use
  PyObject* seq;
  std::vector<void*> at;
  explicit Caches(PyObject* o) : seq(PySequence_Fast(o, "caches must be a sequence of tensors")) {
    if (seq == nullptr) throw python_error();
  }
  ~Caches() { Py_DECREF(seq); }
  size_t size() const { return (size_t)PySequence_Fast_GET_SIZE(seq); }
  const Tensor& operator[](size_t i) const {
    PyObject* o = PySequence_Fast_GET_ITEM(seq, (Py_ssize_t)i);
    Args one{&o, 1};
    return one.tensor();
  }
};

PyObject* py_kv_commit(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  Caches k(a.next()), v(a.next());
  const Tensor* table = a.tensor_or_none();
  const Tensor &path = a.tensor(), &len = a.tensor(), &prefix_len = a.tensor();
  const int32_t N = a.i32();
  const Tensor *out_given = a.tensor_or_none(), *status = a.tensor_or_none();
  PyObject* on_stream = a.next();
  const size_t L = k.size();
  if (L == 0) fail(PyExc_IndexError, "no caches");
  if (v.size() > L) fail(PyExc_IndexError, "more value caches than key caches");
  const Tensor k0 = k[0];
  for (size_t l = 0; l < std::min(L, v.size()); ++l) {
    same_layout(k[l], k0, table != nullptr ? "all layer pools" : "all layer caches");
    same_layout(v[l], k0, table != nullptr ? "all layer pools" : "all layer caches");
  }
  need_dims(k0, 4, "a cache");
  if (table != nullptr) need_dims(*table, 2, "block_table");
  need_dims(path, 2, "accepted_path");
  spec_attn_desc_t d = {};
  const int64_t H = k0.size(1), D = k0.size(3);
  d.B = (int32_t)(table != nullptr ? table->size(0) : k0.size(0));
  d.H = d.H_kv = (int32_t)H;
  d.D = (int32_t)D;
  d.N = N;
  d.S_cap = (int32_t)(table != nullptr ? table->size(1) * k0.size(2) : k0.size(2));
  d.dtype = dtype_code(k0);
  d.q_stride_b = (int64_t)N * H * D; d.q_stride_n = H * D; d.q_stride_h = D;
  d.kv_stride_b = k0.stride(0); d.kv_stride_h = k0.stride(1); d.kv_stride_s = k0.stride(2);
  const Tensor out = out_given != nullptr ? *out_given : empty_as(prefix_len);
  k.at.assign(L, nullptr);
  v.at.assign(L, nullptr);
  for (size_t l = 0; l < L; ++l) k.at[l] = ptr(k[l]);
  for (size_t l = 0; l < v.size(); ++l) v.at[l] = ptr(v[l]);
  const auto *pp = as<int32_t>(path), *lp = as<int32_t>(len), *pl = as<int32_t>(prefix_len);
  int32_t *op = as<int32_t>(out), *st = as<int32_t>(status);
  const int32_t Lmax = (int32_t)path.size(1);
  void* stream = handle(on_stream);
  if (table != nullptr) {
    const spec_kv_pages_t pages = make_pages(k0, *table);
    call("spec_kv_commit_paged", [&] {
      return spec_kv_commit_paged(&d, &pages, (int32_t)L, k.at.data(), v.at.data(), pp, Lmax, lp, pl, op, st, stream); });
  } else {
    call("spec_kv_commit", [&] { return spec_kv_commit(&d, (int32_t)L, k.at.data(), v.at.data(), pp, Lmax, lp, pl, op, st, stream); });
  }
  return wrap(out);
  END_HANDLE_TH_ERRORS
}

// set_helpers(SpecError, ctypes.ArgumentError, _stream)
PyObject* py_set_helpers(PyObject*, PyObject* const* argv, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  Args a{argv, n};
  for (PyObject** to : {&g_spec_error, &g_argument_error, &g_stream}) {
    PyObject* o = a.next();
    Py_INCREF(o);
    Py_XDECREF(*to);
    *to = o;
  }
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

#define SPEC_METHOD(name) {#name, (PyCFunction)(void (*)())py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SPEC_METHOD(set_helpers), SPEC_METHOD(fill_desc), SPEC_METHOD(tree_attention), SPEC_METHOD(verify_greedy), SPEC_METHOD(verify_stochastic),
    SPEC_METHOD(expand_topk), SPEC_METHOD(tree_merge), SPEC_METHOD(lm_head_argmax), SPEC_METHOD(verify_greedy_lm_head),
    SPEC_METHOD(lm_head_logits_stats), SPEC_METHOD(kv_commit), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "spec_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_spec_marshal() { return PyModule_Create(&module); }
