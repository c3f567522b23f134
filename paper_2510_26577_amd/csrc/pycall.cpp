// Python entry points of libtva in native code: what binding.py, verify.py and draft.py would do with ctypes for a
// call on tensors -- read the tensors' shapes and addresses, allocate results and scratch memory, fill the argument
// block, ask for the stream, call the library -- done here on torch's own C++ objects.
//
// Why: a call's kernels take 5 .. 20 us at batch 1, and the interpreter spent longer than that around them
// (tree_verify_attn 23.6 us per call, of which 7.3 the two launches; the stream alone 2.9, three allocations 7, the
// argument block field by field 4).  The library's functions are reached through addresses handed over by bind(), so
// that whichever build of libtva the process has loaded is the one that runs.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/LegacyTypeDispatch.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include "tva.h"
#include "tva_draft.h"
#include "tva_verify.h"

namespace {

// ---- the library's functions, in the order bind() takes their addresses ----
struct Lib {
  int (*attn)(const tva_args *, void *);
  size_t (*workspace_bytes)(const tva_args *);
  int (*mask)(const int32_t *, const int32_t *, int32_t, int32_t, int32_t, uint64_t *, int32_t *, void *);
  int (*greedy)(const int32_t *, const int32_t *, const int32_t *, const int32_t *, int32_t, int32_t, int32_t *, int32_t *, int32_t *,
                void *);
  int (*greedy_filled)(const int32_t *, const int32_t *, const int32_t *, const int32_t *, int32_t, int32_t, int32_t *, int32_t *,
                       int32_t *, void *);
  int (*sampling_filled)(const tva_sample_args *, void *);
  size_t (*sample_workspace)(int32_t, int32_t, int32_t);
  int (*commit)(const tva_commit_args *, void *);
  int (*rerank)(const float *, int32_t, int32_t, const double *, int32_t, double, int32_t *, int32_t *, int32_t *, void *, size_t, void *);
  size_t (*rerank_workspace)(int32_t, int32_t, int32_t);
  int (*subtree)(const float *, const int32_t *, const int32_t *, const int32_t *, int32_t, int32_t, int32_t *, int32_t *, int32_t *,
                 void *);
} lib;
constexpr int kFunctions = sizeof(Lib) / sizeof(void *);

// ---- arguments ----
[[noreturn]] void fail(PyObject *type, const char *message) {
  PyErr_SetString(type, message);
  throw python_error();
}
const at::Tensor *tensor_or_null(PyObject *o) {
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a tensor is expected");
  return &THPVariable_Unpack(o);
}
const at::Tensor &tensor(PyObject *o) {
  const at::Tensor *t = tensor_or_null(o);
  if (!t) fail(PyExc_TypeError, "a tensor is expected, not None");
  return *t;
}
template <class T>
T *ptr(const at::Tensor *t) {
  return t ? static_cast<T *>(t->data_ptr()) : nullptr;
}
int64_t integer(PyObject *o) {
  int64_t v;
  if (PyLong_Check(o)) {
    v = PyLong_AsLongLong(o);
  } else {
    PyObject *n = PyNumber_Long(o);
    if (!n) throw python_error();
    v = PyLong_AsLongLong(n);
    Py_DECREF(n);
  }
  if (v == -1 && PyErr_Occurred()) throw python_error();
  return v;
}
int32_t int32(PyObject *o) { return static_cast<int32_t>(integer(o)); }
double number(PyObject *o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw python_error();
  return v;
}
bool truth(PyObject *o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw python_error();
  return v != 0;
}
void *stream_of(PyObject *o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  PyObject *s = PyObject_GetAttrString(o, "cuda_stream");
  if (!s) throw python_error();
  void *p = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  if (!p && PyErr_Occurred()) throw python_error();
  return p;
}
void strides_of(PyObject *o, int64_t *page, int64_t *tok, int64_t *head) {
  THPObjectPtr seq(PySequence_Fast(o, "strides is a sequence of three numbers"));
  if (!seq) throw python_error();
  if (PySequence_Fast_GET_SIZE(seq.get()) != 3) fail(PyExc_ValueError, "strides is a sequence of three numbers");
  PyObject **v = PySequence_Fast_ITEMS(seq.get());
  *page = integer(v[0]), *tok = integer(v[1]), *head = integer(v[2]);
}
at::Tensor make(at::IntArrayRef sizes, at::ScalarType type, const at::Tensor &like) {
  at::AutoDispatchBelowADInplaceOrView below;
  return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}
// Scratch memory made here comes from the current stream's pool and goes back to it when the call returns.  Work queued
// on another stream still uses it then: the allocator is told, and hands it out again only behind that work.
void hold_for(const at::Tensor &scratch, void *st, PyObject *stream_given) {
  if (!scratch.defined() || stream_given == Py_None) return;
  const auto device = scratch.device().index();
  if (c10::hip::getCurrentHIPStream(device).stream() == st) return;
  c10::hip::HIPCachingAllocator::recordStream(scratch.storage().data_ptr(), c10::hip::getStreamFromExternal(static_cast<hipStream_t>(st), device));
}
int64_t bytes_of(const at::Tensor &t) { return t.numel() * static_cast<int64_t>(t.element_size()); }

// the library's call without the interpreter's lock (as ctypes makes it)
template <class F>
int unlocked(F f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS rc = f();
  Py_END_ALLOW_THREADS return rc;
}
void expect(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) fail(PyExc_TypeError, "wrong number of arguments");
}
PyObject *pair(const at::Tensor &a, const at::Tensor &b) {
  PyObject *t = PyTuple_New(2);
  PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(a));
  PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(b));
  return t;
}
PyObject *triple(const at::Tensor &a, const at::Tensor &b, const at::Tensor &c) {
  PyObject *t = PyTuple_New(3);
  PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(a));
  PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(b));
  PyTuple_SET_ITEM(t, 2, THPVariable_Wrap(c));
  return t;
}

// A host array of int32 (tva_args.L_host), read in place
struct HostInts {
  Py_buffer view{};
  bool held = false;
  const int32_t *data = nullptr;
  HostInts(PyObject *o, int64_t n) {
    if (o == Py_None) return;
    if (PyObject_GetBuffer(o, &view, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) throw python_error();
    held = true;
    if (view.ndim != 1 || view.itemsize != 4 || view.shape[0] != n || !view.format || (view.format[0] != 'i' && view.format[0] != 'l')) {
      PyBuffer_Release(&view);
      held = false;
      fail(PyExc_AssertionError, "L_host is a contiguous array of int32, one per sequence");
    }
    data = static_cast<const int32_t *>(view.buf);
  }
  ~HostInts() {
    if (held) PyBuffer_Release(&view);
  }
};

// Every function below returns its results, or the library's negative status as an int.

// the arguments of binding.tree_verify_attn in order
PyObject *attn(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 30);
  const at::Tensor &q = tensor(a[0]), &cu_T = tensor(a[6]);
  const at::Tensor *k_tree = tensor_or_null(a[1]), *v_tree = tensor_or_null(a[2]), *k_cache = tensor_or_null(a[3]),
                   *v_cache = tensor_or_null(a[4]), *mask = tensor_or_null(a[5]), *L = tensor_or_null(a[7]), *cu_L = tensor_or_null(a[11]),
                   *table = tensor_or_null(a[12]), *out = tensor_or_null(a[16]), *lse = tensor_or_null(a[17]), *ws = tensor_or_null(a[18]),
                   *parent = tensor_or_null(a[20]), *cu_Q = tensor_or_null(a[21]);
  tva_args t{};
  t.B = static_cast<int32_t>(cu_T.numel() - 1);
  t.sum_T = static_cast<int32_t>(q.size(0)), t.Hq = static_cast<int32_t>(q.size(1)), t.D = static_cast<int32_t>(q.size(2));
  t.max_T = int32(a[8]), t.max_L = int32(a[9]);
  t.scale = static_cast<float>(number(a[10]));
  if (cu_Q) {
    t.sum_Q = t.sum_T, t.max_Q = int32(a[22]);
    if (a[23] != Py_None) t.sum_T = int32(a[23]);
    else t.sum_T = static_cast<int32_t>(tensor(a[1]).size(0));
  }
  t.Hkv = static_cast<int32_t>(k_tree ? k_tree->size(1) : tensor(a[3]).size(-2));
  t.mask_words = mask ? static_cast<int32_t>(mask->size(1)) : t.max_T > 64 ? (t.max_T + 63) / 64 : 1;
  t.cu_T = ptr<const int32_t>(&cu_T), t.L = ptr<const int32_t>(L);
  t.q = q.data_ptr(), t.k_tree = ptr<void>(k_tree), t.v_tree = ptr<void>(v_tree), t.anc_mask = ptr<const uint64_t>(mask);
  t.k_cache = ptr<void>(k_cache), t.v_cache = ptr<void>(v_cache);
  t.cu_L = ptr<const int32_t>(cu_L), t.page_table = ptr<const int32_t>(table), t.cu_Q = ptr<const int32_t>(cu_Q);
  t.parent = ptr<const int32_t>(parent);
  t.page_size = int32(a[13]);
  t.max_pages = table ? static_cast<int32_t>(table->size(1)) : 0;
  strides_of(a[14], &t.stride_page, &t.stride_tok, &t.stride_head);
  t.num_splits = int32(a[15]);
  t.kv_fp8 = truth(a[24]);
  t.k_scale = static_cast<float>(number(a[25])), t.v_scale = static_cast<float>(number(a[26]));
  t.sum_L = integer(a[27]);
  t.plan_shape = int32(a[28]);
  const HostInts lengths(a[29], t.B);
  t.L_host = lengths.data;
  at::Tensor new_out, new_lse, new_ws;
  if (!out) new_out = make(q.sizes(), at::kFloat, q), out = &new_out;
  if (!lse) new_lse = make({q.size(0), q.size(1)}, at::kFloat, q), lse = &new_lse;
  t.out = ptr<float>(out), t.lse = ptr<float>(lse);
  const size_t need = lib.workspace_bytes(&t);
  if (need == (size_t)-1) return PyLong_FromLong(TVA_INVALID_ARG);
  if (need > 0 && (!ws || (size_t)bytes_of(*ws) < need)) new_ws = make({(int64_t)((need + 3) / 4)}, at::kFloat, q), ws = &new_ws;
  if (ws) t.workspace = ws->data_ptr(), t.workspace_bytes = (size_t)bytes_of(*ws);
  void *st = stream_of(a[19]);
  const int rc = unlocked([&] { return lib.attn(&t, st); });
  hold_for(new_ws, st, a[19]);
  if (rc != TVA_OK) return PyLong_FromLong(rc);
  return pair(*out, *lse);
  END_HANDLE_TH_ERRORS
}

// (parent, cu_T, max_T, mask, err_flag, stream)
PyObject *ancestor_mask(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 6);
  const at::Tensor &parent = tensor(a[0]), &cu_T = tensor(a[1]);
  const at::Tensor *mask = tensor_or_null(a[3]), *flag = tensor_or_null(a[4]);
  const int32_t max_T = int32(a[2]);
  const int32_t W = mask ? static_cast<int32_t>(mask->size(1)) : max_T > 64 ? (max_T + 63) / 64 : 1;
  at::Tensor made;
  if (!mask) made = make({parent.numel(), W}, at::kLong, parent), mask = &made;
  void *st = stream_of(a[5]);
  const int rc = unlocked([&] {
    return lib.mask(ptr<const int32_t>(&parent), ptr<const int32_t>(&cu_T), static_cast<int32_t>(cu_T.numel() - 1), max_T, W,
                    ptr<uint64_t>(mask), ptr<int32_t>(flag), st);
  });
  if (rc != TVA_OK) return PyLong_FromLong(rc);
  return THPVariable_Wrap(*mask);
  END_HANDLE_TH_ERRORS
}

// (parent, cu_T, draft_token, target_token, max_path, path, path_len, next_token, stream)
PyObject *accept_greedy(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 9);
  const at::Tensor &parent = tensor(a[0]), &cu_T = tensor(a[1]), &draft = tensor(a[2]), &target = tensor(a[3]);
  const at::Tensor *path = tensor_or_null(a[5]), *len = tensor_or_null(a[6]), *next = tensor_or_null(a[7]);
  const int64_t B = cu_T.numel() - 1, max_path = integer(a[4]);
  at::Tensor new_path, new_len, new_next;
  const bool fill = !path;  // (a path made here has -1 behind the accepted nodes)
  if (!path) new_path = make({B, max_path}, at::kInt, cu_T), path = &new_path;
  if (!len) new_len = make({B}, at::kInt, cu_T), len = &new_len;
  if (!next) new_next = make({B}, at::kInt, cu_T), next = &new_next;
  void *st = stream_of(a[8]);
  const int rc = unlocked([&] {
    return (fill ? lib.greedy_filled : lib.greedy)(ptr<const int32_t>(&parent), ptr<const int32_t>(&cu_T), ptr<const int32_t>(&draft),
                                                   ptr<const int32_t>(&target), (int32_t)B, (int32_t)max_path, ptr<int32_t>(path),
                                                   ptr<int32_t>(len), ptr<int32_t>(next), st);
  });
  if (rc != TVA_OK) return PyLong_FromLong(rc);
  return triple(*path, *len, *next);
  END_HANDLE_TH_ERRORS
}

// (parent, cu_T, draft_token, p_target, q_draft, u, u_final, max_path, residual, err_flag, stream, workspace or None,
//  make a workspace, workgroups_per_sequence, sum_T, unit_rows)
PyObject *accept_sampling(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 16);
  const at::Tensor &cu_T = tensor(a[1]), &p = tensor(a[3]);
  const at::Tensor *residual = tensor_or_null(a[8]), *ws = tensor_or_null(a[11]);
  tva_sample_args t{};
  const int64_t B = cu_T.numel() - 1, V = p.size(1), max_path = integer(a[7]);
  t.B = (int32_t)B, t.V = (int32_t)V, t.max_path = (int32_t)max_path;
  t.workgroups_per_sequence = int32(a[13]), t.sum_T = int32(a[14]), t.unit_rows = truth(a[15]);
  at::Tensor path = make({B, max_path}, at::kInt, cu_T), len = make({B}, at::kInt, cu_T), next = make({B}, at::kInt, cu_T), made, made_ws;
  if (!residual) made = make({B > 1 ? B : 1, V}, at::kFloat, cu_T), residual = &made;
  if (!ws && truth(a[12])) {
    const size_t need = lib.sample_workspace(t.B, t.sum_T, t.V) / 8;
    made_ws = make({(int64_t)(need > 1 ? need : 1)}, at::kLong, cu_T), ws = &made_ws;
  }
  t.parent = ptr<const int32_t>(tensor_or_null(a[0])), t.cu_T = ptr<const int32_t>(&cu_T);
  t.draft_token = ptr<const int32_t>(tensor_or_null(a[2]));
  t.p_target = ptr<const float>(&p), t.q_draft = ptr<const float>(tensor_or_null(a[4]));
  t.u = ptr<const float>(tensor_or_null(a[5])), t.u_final = ptr<const float>(tensor_or_null(a[6]));
  t.residual = ptr<float>(residual), t.err_flag = ptr<int32_t>(tensor_or_null(a[9]));
  t.path = ptr<int32_t>(&path), t.path_len = ptr<int32_t>(&len), t.next_token = ptr<int32_t>(&next);
  if (ws) t.workspace = ws->data_ptr(), t.workspace_bytes = (size_t)bytes_of(*ws);
  void *st = stream_of(a[10]);
  const int rc = unlocked([&] { return lib.sampling_filled(&t, st); });
  hold_for(made, st, a[10]);
  hold_for(made_ws, st, a[10]);
  if (rc != TVA_OK) return PyLong_FromLong(rc);
  return triple(path, len, next);
  END_HANDLE_TH_ERRORS
}

// the arguments of verify.make_commit_args in order, and the stream
PyObject *commit_path(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 18);
  const at::Tensor &cu_T = tensor(a[0]), &path = tensor(a[2]), &kc = tensor(a[6]);
  tva_commit_args t{};
  t.B = static_cast<int32_t>(cu_T.numel() - 1);
  t.Hkv = static_cast<int32_t>(kc.size(-2)), t.D = static_cast<int32_t>(kc.size(-1)), t.max_path = static_cast<int32_t>(path.size(1));
  t.cu_T = ptr<const int32_t>(&cu_T), t.L = ptr<const int32_t>(tensor_or_null(a[1])), t.path = ptr<const int32_t>(&path);
  t.path_len = ptr<const int32_t>(tensor_or_null(a[3]));
  t.k_tree = ptr<void>(tensor_or_null(a[4])), t.v_tree = ptr<void>(tensor_or_null(a[5]));
  t.k_cache = kc.data_ptr(), t.v_cache = ptr<void>(tensor_or_null(a[7]));
  const at::Tensor *table = tensor_or_null(a[9]);
  t.cu_L = ptr<const int32_t>(tensor_or_null(a[8])), t.page_table = ptr<const int32_t>(table);
  t.page_size = int32(a[10]), t.max_pages = table ? static_cast<int32_t>(table->size(1)) : 0;
  strides_of(a[11], &t.stride_page, &t.stride_tok, &t.stride_head);
  t.L_out = ptr<int32_t>(tensor_or_null(a[12])), t.err_flag = ptr<int32_t>(tensor_or_null(a[13]));
  t.n_layers = int32(a[14]), t.layer_stride_cache = integer(a[15]), t.layer_stride_tree = integer(a[16]);
  if (kc.element_size() == 1) {
    // 8-bit K/V: the kernels only move bytes, so a row of D bytes is passed as D / 2 two-byte elements
    if ((t.D | t.stride_page | t.stride_tok | t.stride_head | t.layer_stride_cache | t.layer_stride_tree) & 1)
      fail(PyExc_ValueError, "8-bit K/V: D and the strides are even");
    t.D /= 2, t.stride_page /= 2, t.stride_tok /= 2, t.stride_head /= 2, t.layer_stride_cache /= 2, t.layer_stride_tree /= 2;
  }
  void *st = stream_of(a[17]);
  return PyLong_FromLong(unlocked([&] { return lib.commit(&t, st); }));
  END_HANDLE_TH_ERRORS
}

// (tree_scores, cost_row, m, C3, count, cu_T, err_flag, stream, workspace)
PyObject *rerank_count(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 9);
  const at::Tensor &scores = tensor(a[0]), &cost = tensor(a[1]);
  const at::Tensor *count = tensor_or_null(a[4]), *cu_T = tensor_or_null(a[5]), *flag = tensor_or_null(a[6]), *ws = tensor_or_null(a[8]);
  const int32_t B = (int32_t)scores.size(0), N = (int32_t)scores.size(1), m = int32(a[2]);
  const double C3 = number(a[3]);
  at::Tensor new_count, new_cu, new_ws;
  if (!count) new_count = make({1}, at::kInt, scores), count = &new_count;
  if (!cu_T) new_cu = make({B + 1}, at::kInt, scores), cu_T = &new_cu;
  if (!ws) {
    const size_t need = lib.rerank_workspace(B, N, m);
    if (need == (size_t)-1) return PyLong_FromLong(TVA_INVALID_ARG);
    new_ws = make({(int64_t)(need / 4 > 1 ? need / 4 : 1)}, at::kFloat, scores), ws = &new_ws;
  }
  void *st = stream_of(a[7]);
  const int rc = unlocked([&] {
    return lib.rerank(ptr<const float>(&scores), B, N, ptr<const double>(&cost), m, C3, ptr<int32_t>(count), ptr<int32_t>(cu_T),
                      ptr<int32_t>(flag), ws->data_ptr(), (size_t)bytes_of(*ws), st);
  });
  hold_for(new_ws, st, a[7]);
  if (rc != TVA_OK) return PyLong_FromLong(rc);
  return pair(*count, *cu_T);
  END_HANDLE_TH_ERRORS
}

// (score, parent, cu_M, cu_T, max_M, old_index, new_parent, err_flag, stream, total_kept)
PyObject *select_subtree(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 10);
  const at::Tensor &score = tensor(a[0]), &parent = tensor(a[1]), &cu_M = tensor(a[2]), &cu_T = tensor(a[3]);
  const at::Tensor *old_index = tensor_or_null(a[5]), *new_parent = tensor_or_null(a[6]), *flag = tensor_or_null(a[7]);
  at::Tensor new_old, new_new;
  if (!old_index || !new_parent) {
    const int64_t kept = integer(a[9]) > 1 ? integer(a[9]) : 1;
    if (!old_index) new_old = make({kept}, at::kInt, score), old_index = &new_old;
    if (!new_parent) new_new = make({kept}, at::kInt, score), new_parent = &new_new;
  }
  const int32_t max_M = int32(a[4]);
  void *st = stream_of(a[8]);
  const int rc = unlocked([&] {
    return lib.subtree(ptr<const float>(&score), ptr<const int32_t>(&parent), ptr<const int32_t>(&cu_M), ptr<const int32_t>(&cu_T),
                       (int32_t)(cu_M.numel() - 1), max_M, ptr<int32_t>(old_index), ptr<int32_t>(new_parent), ptr<int32_t>(flag), st);
  });
  if (rc != TVA_OK) return PyLong_FromLong(rc);
  return pair(*old_index, *new_parent);
  END_HANDLE_TH_ERRORS
}

// A call on an argument block the caller keeps: (address of int f(const void *args, void *stream), how many bytes f reads
// of the block, the block's class, the block, stream) -> status.  Another structure is refused: f would take its fields
// for its own, and read past a shorter one's end.
PyObject *call(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 5);
  auto f = reinterpret_cast<int (*)(const void *, void *)>(PyLong_AsVoidPtr(a[0]));
  if (!f) fail(PyExc_ValueError, "the function has no address");
  const int64_t size = integer(a[1]);
  const int right = PyObject_IsInstance(a[3], a[2]);
  if (right < 0) throw python_error();
  if (!right) {
    PyErr_Format(PyExc_TypeError, "expected %S, not %S", a[2], reinterpret_cast<PyObject *>(Py_TYPE(a[3])));
    throw python_error();
  }
  struct Block {
    Py_buffer view{};
    explicit Block(PyObject *o) {
      if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) throw python_error();
    }
    ~Block() { PyBuffer_Release(&view); }
  } block(a[3]);
  if (block.view.len < size) fail(PyExc_TypeError, "the argument block is shorter than the library's");
  void *st = stream_of(a[4]);
  return PyLong_FromLong(unlocked([&] { return f(block.view.buf, st); }));
  END_HANDLE_TH_ERRORS
}

// (stream or None) -> the stream's address
PyObject *stream(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, 1);
  return PyLong_FromVoidPtr(stream_of(a[0]));
  END_HANDLE_TH_ERRORS
}

// the addresses of the library's functions, in the order of `Lib`
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  expect(n, kFunctions);
  void *at[kFunctions];
  for (int i = 0; i < kFunctions; ++i) {
    at[i] = PyLong_AsVoidPtr(a[i]);
    if (!at[i]) fail(PyExc_ValueError, "a function has no address");
  }
  memcpy(&lib, at, sizeof(lib));
  Py_RETURN_NONE;
  END_HANDLE_TH_ERRORS
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr
PyMethodDef methods[] = {{"attn", FAST(attn)},
                         {"ancestor_mask", FAST(ancestor_mask)},
                         {"accept_greedy", FAST(accept_greedy)},
                         {"accept_sampling", FAST(accept_sampling)},
                         {"commit_path", FAST(commit_path)},
                         {"rerank_count", FAST(rerank_count)},
                         {"select_subtree", FAST(select_subtree)},
                         {"call", FAST(call)},
                         {"stream", FAST(stream)},
                         {"bind", FAST(bind)},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall(void) {
  PyObject *m = PyModule_Create(&module);
  if (!m) return nullptr;
  PyModule_AddIntConstant(m, "functions", kFunctions);
  // the argument blocks this module fills must be the ones the loaded library reads
  PyModule_AddIntConstant(m, "sizes", (long)(sizeof(tva_args) + 1024 * (sizeof(tva_sample_args) + 1024 * sizeof(tva_commit_args))));
  return m;
}
