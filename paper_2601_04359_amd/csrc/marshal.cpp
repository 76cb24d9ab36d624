// Native marshalling of the binding's calls: what binding.py does with ctypes, for plain arguments.
//
// A small call spends most of its time on the host (one frame step of a small layer: 36 us of kernels behind 60 us
// of Python and launches), and a ctypes call with twenty arguments and the tensor queries in front of it cost 5 to
// 10 us.  Here the same checks and the same library call take under 1.  Arguments that are not plain (strided GPU
// tensors, built-in integers in 32-bit range, lists and tuples of them), and calls that the checks would refuse,
// return None: binding.py then takes its own path, which converts, or raises with the message.  The library's
// status comes back as an integer.  The entry points' addresses come from binding.py (bind), so both paths
// call the same loaded library.  The interpreter's lock is released around every library call.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/TensorBody.h>
#include <ATen/ops/empty.h>

#include <limits.h>
#include <stdint.h>

#include <vector>

#include "packcache.h"

namespace {

struct Library {
  decltype(&pc_rope3d) rope3d;
  decltype(&pc_score) score;
  decltype(&pc_compact) compact;
  decltype(&pc_compact_batch) compact_batch;
  decltype(&pc_frame_attn) frame_attn;
  decltype(&pc_frame_attn_workspace_bytes_for) attn_bytes;
  decltype(&pc_budget) budget;
} lib = {};
PyObject* current_device = nullptr;   // torch's raw queries of the current device and of its stream
PyObject* raw_stream = nullptr;

// The lock comes back on every way out: an exception's way leads to a Python error.
template <class F>
auto unlocked(F&& call) {
  struct Lock {
    PyThreadState* state = PyEval_SaveThread();
    ~Lock() { PyEval_RestoreThread(state); }
  } lock;
  return call();
}

// ---- plain arguments -------------------------------------------------------------------------
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchGradWrapper,
                                         c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::Functionalize,
                                         c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                         c10::DispatchKey::ZeroTensor});
  if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || t.key_set().has_any(wrapped)) return nullptr;
  return &t;
}
// rows dense, last dimension contiguous
bool rows_dense(const at::Tensor& t, int64_t dim) {
  return t.dim() == dim && t.stride(dim - 1) == 1 && t.stride(dim - 2) == t.size(dim - 1);
}
int dtype_code(const at::Tensor& t) {
  return t.scalar_type() == at::kFloat ? PC_F32 : t.scalar_type() == at::kBFloat16 ? PC_BF16 : -1;
}
bool as_int(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  const long long x = PyLong_AsLongLongAndOverflow(o, &over);
  if (over != 0 || x < INT32_MIN || x > INT32_MAX) return false;
  *v = static_cast<int32_t>(x);
  return true;
}
bool size_as_int(int64_t x, int* v) {
  *v = static_cast<int>(x);
  return x >= 0 && x <= INT32_MAX;
}
bool as_double(PyObject* o, double* v) {
  int32_t i;
  if (PyFloat_CheckExact(o)) {
    *v = PyFloat_AS_DOUBLE(o);
    return true;
  }
  if (!as_int(o, &i)) return false;
  *v = i;
  return true;
}
bool as_flag(PyObject* o, int* v) {
  *v = o == Py_True;
  return o == Py_True || o == Py_False;
}
bool is_table(PyObject* o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); }
bool as_ints(PyObject* o, Py_ssize_t n, std::vector<int32_t>& v) {
  if (!is_table(o) || PySequence_Fast_GET_SIZE(o) != n) return false;
  v.resize(n);
  for (Py_ssize_t i = 0; i < n; ++i)
    if (!as_int(PySequence_Fast_GET_ITEM(o, i), &v[i])) return false;
  return true;
}
bool as_segments(PyObject* o, std::vector<pc_segment>& v) {
  if (!is_table(o)) return false;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
  v.resize(n);
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* s = PySequence_Fast_GET_ITEM(o, i);
    if (!is_table(s) || PySequence_Fast_GET_SIZE(s) != 4) return false;
    int32_t f[4];
    for (int k = 0; k < 4; ++k)
      if (!as_int(PySequence_Fast_GET_ITEM(s, k), &f[k])) return false;
    v[i] = {f[0], f[1], f[2], f[3]};
  }
  return n > 0;
}
PyObject* ints(const int32_t* v, Py_ssize_t n) {
  PyObject* list = PyList_New(n);
  for (Py_ssize_t i = 0; list && i < n; ++i) {
    PyObject* x = PyLong_FromLong(v[i]);
    if (!x) {
      Py_DECREF(list);
      return nullptr;
    }
    PyList_SET_ITEM(list, i, x);
  }
  return list;
}
// the current stream of the current device: what a launch without a stream argument would use
bool current_stream(void** out) {
  PyObject* device = PyObject_CallNoArgs(current_device);
  PyObject* handle = device ? PyObject_CallOneArg(raw_stream, device) : nullptr;
  Py_XDECREF(device);
  if (!handle) return false;
  *out = PyLong_AsVoidPtr(handle);
  Py_DECREF(handle);
  return !PyErr_Occurred();
}
// unbound, or a mode that wants to see every tensor method
bool ready() { return raw_stream != nullptr && !at::impl::torch_function_mode_enabled(); }

#define PLAIN_OR_NONE(cond) \
  if (!(cond)) Py_RETURN_NONE

// ---- calls: in the order of binding.py, positional ---------------------------------------------
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {   // 7 addresses, the two queries
  if (n != 9) {
    PyErr_SetString(PyExc_TypeError, "bind: 9 arguments");
    return nullptr;
  }
  void* p[7];
  for (int i = 0; i < 7; ++i) p[i] = PyLong_AsVoidPtr(a[i]);
  if (PyErr_Occurred()) return nullptr;
  lib = {reinterpret_cast<decltype(&pc_rope3d)>(p[0]),
         reinterpret_cast<decltype(&pc_score)>(p[1]),
         reinterpret_cast<decltype(&pc_compact)>(p[2]),
         reinterpret_cast<decltype(&pc_compact_batch)>(p[3]),
         reinterpret_cast<decltype(&pc_frame_attn)>(p[4]),
         reinterpret_cast<decltype(&pc_frame_attn_workspace_bytes_for)>(p[5]),
         reinterpret_cast<decltype(&pc_budget)>(p[6])};
  Py_INCREF(a[7]);
  Py_INCREF(a[8]);
  Py_XSETREF(current_device, a[7]);
  Py_XSETREF(raw_stream, a[8]);
  Py_RETURN_NONE;
}

PyObject* rope3d(PyObject*, PyObject* const* a, Py_ssize_t n_args) {   // x, pos, sections, base, out_scale
  HANDLE_TH_ERRORS
  PLAIN_OR_NONE(n_args == 5 && ready());
  const at::Tensor *x = plain(a[0]), *pos = plain(a[1]);
  PLAIN_OR_NONE(x && pos && rows_dense(*x, 3) && is_table(a[2]) && PySequence_Fast_GET_SIZE(a[2]) >= 3);
  int32_t sec[3];
  for (int i = 0; i < 3; ++i) PLAIN_OR_NONE(as_int(PySequence_Fast_GET_ITEM(a[2], i), &sec[i]));
  double base, out_scale;
  int H, n, D;
  const int dt = dtype_code(*x);
  PLAIN_OR_NONE(dt >= 0 && as_double(a[3], &base) && as_double(a[4], &out_scale) && size_as_int(x->size(0), &H) &&
                size_as_int(x->size(1), &n) && size_as_int(x->size(2), &D));
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  void *xp = x->mutable_data_ptr(), *pp = pos->mutable_data_ptr();
  const int64_t stride = x->stride(0);
  return PyLong_FromLong(unlocked([&] {
    return lib.rope3d(xp, dt, H, n, D, stride, static_cast<int32_t*>(pp), sec[0], sec[1], sec[2], base, out_scale, stream);
  }));
  END_HANDLE_TH_ERRORS
}

// Qs, K, Nk, scale, lse, score, share_heads, ws, q_rows, key_range
PyObject* score(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  PLAIN_OR_NONE(n_args == 10 && ready());
  const at::Tensor *Q = plain(a[0]), *K = plain(a[1]), *out = plain(a[5]), *ws = plain(a[7]);
  const at::Tensor *lse = nullptr, *rows = nullptr;
  PLAIN_OR_NONE(Q && K && out && ws && rows_dense(*Q, 3) && rows_dense(*K, 3) && out->dim() >= 1);
  PLAIN_OR_NONE(a[4] == Py_None || ((lse = plain(a[4])) && lse->dim() >= 1));
  PLAIN_OR_NONE(a[8] == Py_None || (rows = plain(a[8])));
  int32_t Nk, begin = 0, end = 0;
  double scale;
  int share, Hq, Hkv, n_qs, D;
  const int dt = dtype_code(*K);
  PLAIN_OR_NONE(dt >= 0 && as_int(a[2], &Nk) && as_double(a[3], &scale) && as_flag(a[6], &share) &&
                size_as_int(Q->size(0), &Hq) && size_as_int(K->size(0), &Hkv) && size_as_int(Q->size(2), &D) &&
                size_as_int(rows ? rows->numel() : Q->size(1), &n_qs));
  if (a[9] != Py_None)
    PLAIN_OR_NONE(is_table(a[9]) && PySequence_Fast_GET_SIZE(a[9]) >= 2 &&
                  as_int(PySequence_Fast_GET_ITEM(a[9], 0), &begin) && as_int(PySequence_Fast_GET_ITEM(a[9], 1), &end));
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  void *qp = Q->mutable_data_ptr(), *kp = K->mutable_data_ptr(), *op = out->mutable_data_ptr(), *wp = ws->mutable_data_ptr();
  void *lp = lse ? lse->mutable_data_ptr() : nullptr, *rp = rows ? rows->mutable_data_ptr() : nullptr;
  const int64_t qs = Q->stride(0), ks = K->stride(0), os = out->stride(0), ls = lse ? lse->stride(0) : 0;
  const size_t wn = ws->numel();
  return PyLong_FromLong(unlocked([&] {
    return lib.score(qp, kp, dt, Hq, Hkv, n_qs, Nk, D, qs, ks, static_cast<int32_t*>(rp), static_cast<float>(scale),
                     static_cast<float*>(lp), ls, static_cast<float*>(op), os, share, begin, end, wp, wn, stream);
  }));
  END_HANDLE_TH_ERRORS
}

// What _check_kv_layout accepts, for one set of tensors ([L][H][cap][D] with layers, else [H][cap][D]).
bool cache_layout(const at::Tensor& K, const at::Tensor& V, const at::Tensor& pos, int64_t dim, bool share) {
  if (!rows_dense(K, dim) || !rows_dense(V, dim) || !rows_dense(pos, dim) || V.sizes() != K.sizes()) return false;
  for (int64_t i = 0; i < dim - 2; ++i)
    if (V.stride(i) != K.stride(i)) return false;
  return pos.size(dim - 1) == 3 && pos.size(dim - 3) == (share ? 1 : K.size(dim - 3));
}

// K, V, pos, score, segments, budgets, share_heads, out, idx, ws; the caches with a layer axis or without
PyObject* compact_call(PyObject* const* a, Py_ssize_t n_args, bool layers) {
  PLAIN_OR_NONE(n_args == 10 && ready());
  const int64_t dim = layers ? 4 : 3, head = dim - 3;
  const at::Tensor *K = plain(a[0]), *V = plain(a[1]), *pos = plain(a[2]), *sc = plain(a[3]), *ws = plain(a[9]);
  int share;
  PLAIN_OR_NONE(K && V && pos && sc && ws && as_flag(a[6], &share) && cache_layout(*K, *V, *pos, dim, share) &&
                sc->dim() > head);
  const at::Tensor *Ko = K, *Vo = V, *po = pos, *idx = nullptr;
  if (a[7] != Py_None) {
    PLAIN_OR_NONE(PyTuple_CheckExact(a[7]) && PyTuple_GET_SIZE(a[7]) == 3);
    Ko = plain(PyTuple_GET_ITEM(a[7], 0)), Vo = plain(PyTuple_GET_ITEM(a[7], 1)), po = plain(PyTuple_GET_ITEM(a[7], 2));
    PLAIN_OR_NONE(Ko && Vo && po && rows_dense(*Ko, dim) && rows_dense(*Vo, dim) && rows_dense(*po, dim) &&
                  Vo->sizes() == Ko->sizes() && po->size(dim - 1) == 3 && po->size(head) == (share ? 1 : K->size(head)));
    for (int64_t i = 0; i <= head; ++i) PLAIN_OR_NONE(Vo->stride(i) == Ko->stride(i));
  }
  PLAIN_OR_NONE(a[8] == Py_None || ((idx = plain(a[8])) && idx->dim() > head));
  std::vector<pc_segment> seg;
  std::vector<int32_t> budget;
  int L = 1, Hkv, D;
  const int dt = dtype_code(*K);
  PLAIN_OR_NONE(as_segments(a[4], seg) && as_ints(a[5], static_cast<Py_ssize_t>(seg.size()), budget) && dt >= 0 &&
                size_as_int(K->size(head), &Hkv) && size_as_int(K->size(dim - 1), &D) &&
                (!layers || size_as_int(K->size(0), &L)));
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  auto ptr = [](const at::Tensor* t) { return t ? t->mutable_data_ptr() : nullptr; };
  auto by_head = [&](const at::Tensor* t) { return t ? t->stride(head) : 0; };
  auto by_layer = [&](const at::Tensor* t) { return t && layers ? t->stride(0) : 0; };
  void *kp = ptr(K), *vp = ptr(V), *kop = ptr(Ko), *vop = ptr(Vo), *wp = ptr(ws);
  auto *pp = static_cast<int32_t*>(ptr(pos)), *pop = static_cast<int32_t*>(ptr(po)), *ip = static_cast<int32_t*>(ptr(idx));
  auto* sp = static_cast<float*>(ptr(sc));
  const size_t wn = ws->numel();
  const int n = static_cast<int>(seg.size());
  std::vector<pc_segment> seg_out(n);
  int32_t nk = 0;
  const int status = unlocked([&] {
    return layers ? lib.compact_batch(L, kp, vp, pp, dt, Hkv, D, by_head(K), by_layer(K), by_head(pos), by_layer(pos), sp,
                                      by_head(sc), by_layer(sc), seg.data(), n, budget.data(), share, kop, vop, pop,
                                      by_head(Ko), by_layer(Ko), by_head(po), by_layer(po), ip, by_head(idx), by_layer(idx),
                                      seg_out.data(), &nk, wp, wn, stream)
                  : lib.compact(kp, vp, pp, dt, Hkv, D, by_head(K), by_head(pos), sp, by_head(sc), seg.data(), n,
                                budget.data(), share, kop, vop, pop, by_head(Ko), by_head(po), ip, by_head(idx),
                                seg_out.data(), &nk, wp, wn, stream);
  });
  if (status != PC_OK) return PyLong_FromLong(status);
  PyObject* table = PyList_New(n);
  for (int i = 0; table && i < n; ++i) {
    PyObject* s = Py_BuildValue("(iiii)", seg_out[i].start, seg_out[i].len, seg_out[i].kind, seg_out[i].frame);
    if (!s) Py_CLEAR(table);
    else PyList_SET_ITEM(table, i, s);
  }
  return table ? Py_BuildValue("(Ni)", table, nk) : nullptr;
}
PyObject* compact(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  return compact_call(a, n, false);
  END_HANDLE_TH_ERRORS
}
PyObject* compact_batch(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  return compact_call(a, n, true);
  END_HANDLE_TH_ERRORS
}

PyObject* frame_attn(PyObject*, PyObject* const* a, Py_ssize_t n_args) {   // Q, K, V, Nk, scale, O, lse, ws
  HANDLE_TH_ERRORS
  PLAIN_OR_NONE(n_args == 8 && ready());
  const at::Tensor *Q = plain(a[0]), *K = plain(a[1]), *V = plain(a[2]), *O = plain(a[5]), *lse = nullptr, *ws = nullptr;
  PLAIN_OR_NONE(Q && K && V && O && rows_dense(*Q, 3) && rows_dense(*K, 3) && rows_dense(*V, 3) &&
                K->stride(0) == V->stride(0) && O->dim() >= 1);
  int32_t Nk;
  double scale;
  int Hq, Hkv, Nq, D;
  const int dt = dtype_code(*Q);
  PLAIN_OR_NONE(dt >= 0 && as_int(a[3], &Nk) && as_double(a[4], &scale) && size_as_int(Q->size(0), &Hq) &&
                size_as_int(K->size(0), &Hkv) && size_as_int(Q->size(1), &Nq) && size_as_int(Q->size(2), &D));
  PLAIN_OR_NONE(a[6] == Py_None || ((lse = plain(a[6])) && lse->dim() == 2 && lse->size(0) == Hq && lse->size(1) == Nq &&
                                    lse->is_contiguous()));
  PLAIN_OR_NONE(a[7] == Py_None || (ws = plain(a[7])));
  at::Tensor own;   // a workspace of the call's own, from torch's stream-ordered allocator
  if (!ws) {
    const size_t bytes = lib.attn_bytes(dt, Hq, Hkv, Nq, Nk, D);
    if (bytes) {
      own = at::empty({static_cast<int64_t>(bytes < 16 ? 16 : bytes)},
                      at::TensorOptions().dtype(at::kByte).device(Q->device()));
      ws = &own;
    }
  }
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  void *qp = Q->mutable_data_ptr(), *kp = K->mutable_data_ptr(), *vp = V->mutable_data_ptr(), *op = O->mutable_data_ptr();
  void *lp = lse ? lse->mutable_data_ptr() : nullptr, *wp = ws ? ws->mutable_data_ptr() : nullptr;
  const int64_t qs = Q->stride(0), ks = K->stride(0), os = O->stride(0);
  const size_t wn = ws ? ws->numel() : 0;
  return PyLong_FromLong(unlocked([&] {
    return lib.frame_attn(qp, kp, vp, dt, Hq, Hkv, Nq, Nk, D, qs, ks, os, static_cast<float>(scale), op,
                          static_cast<float*>(lp), wp, wn, stream);
  }));
  END_HANDLE_TH_ERRORS
}

// Rows start .. start + n - 1 of three caches as views: K, V, pos, dim, start, n
PyObject* rows(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  PLAIN_OR_NONE(n_args == 6 && ready());
  int32_t dim, start, n;
  PLAIN_OR_NONE(as_int(a[3], &dim) && as_int(a[4], &start) && as_int(a[5], &n) && dim >= 0 && start >= 0 && n >= 0);
  const at::Tensor* t[3];
  for (int i = 0; i < 3; ++i)
    PLAIN_OR_NONE((t[i] = plain(a[i])) && t[i]->dim() > dim && static_cast<int64_t>(start) + n <= t[i]->size(dim));
  PyObject* views = PyTuple_New(3);
  for (int i = 0; views && i < 3; ++i) {
    PyObject* v = THPVariable_Wrap(t[i]->narrow(dim, start, n));
    if (!v) Py_CLEAR(views);
    else PyTuple_SET_ITEM(views, i, v);
  }
  return views;
  END_HANDLE_TH_ERRORS
}

// ---- tables (host only) ------------------------------------------------------------------------
PyObject* budget(PyObject*, PyObject* const* a, Py_ssize_t n_args) {   // mode, n_frame_tokens, n_past, gamma, b_min
  HANDLE_TH_ERRORS
  int32_t mode, n, n_past, b_min;
  double gamma;
  PLAIN_OR_NONE(n_args == 5 && lib.budget && as_int(a[0], &mode) && as_int(a[1], &n) && as_int(a[2], &n_past) &&
                as_double(a[3], &gamma) && as_int(a[4], &b_min) && n_past >= 0 && n_past <= 1 << 16);
  std::vector<int32_t> out(n_past + 1);
  const int status = lib.budget(mode, n, n_past, gamma, b_min, out.data());
  return status != PC_OK ? PyLong_FromLong(status) : ints(out.data(), n_past);
  END_HANDLE_TH_ERRORS
}

PyObject* segment_budgets(PyObject*, PyObject* const* a, Py_ssize_t n_args) {   // segments, by_distance
  HANDLE_TH_ERRORS
  std::vector<pc_segment> seg;
  PLAIN_OR_NONE(n_args == 2 && as_segments(a[0], seg) && is_table(a[1]));
  const Py_ssize_t n_by = PySequence_Fast_GET_SIZE(a[1]);
  std::vector<int32_t> out(seg.size());
  Py_ssize_t d = 0;
  for (size_t i = seg.size(); i-- > 0;) {
    out[i] = seg[i].len;
    if (seg[i].kind != PC_SEG_FRAME) continue;
    PLAIN_OR_NONE(d < n_by && as_int(PySequence_Fast_GET_ITEM(a[1], d), &out[i]));
    ++d;
  }
  return ints(out.data(), static_cast<Py_ssize_t>(out.size()));
  END_HANDLE_TH_ERRORS
}

// How many past frames a table holds: segments
PyObject* past_frames(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  std::vector<pc_segment> seg;
  PLAIN_OR_NONE(n_args == 1 && as_segments(a[0], seg));
  long n = 0;
  for (const pc_segment& s : seg) n += s.kind == PC_SEG_FRAME;
  return PyLong_FromLong(n);
  END_HANDLE_TH_ERRORS
}

// Rows from the first to the last past frame that is over its budget, False if none is: segments, budgets
PyObject* prunable_span(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  std::vector<pc_segment> seg;
  std::vector<int32_t> b;
  PLAIN_OR_NONE(n_args == 2 && as_segments(a[0], seg) && as_ints(a[1], static_cast<Py_ssize_t>(seg.size()), b));
  int64_t begin = -1, end = 0;
  for (size_t i = 0; i < seg.size(); ++i)
    if (seg[i].kind == PC_SEG_FRAME && b[i] < seg[i].len) {
      if (begin < 0) begin = seg[i].start;
      end = static_cast<int64_t>(seg[i].start) + seg[i].len;
    }
  if (begin < 0) Py_RETURN_FALSE;
  return Py_BuildValue("(LL)", static_cast<long long>(begin), static_cast<long long>(end));
  END_HANDLE_TH_ERRORS
}

#define ENTRY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(bind),       ENTRY(rope3d),      ENTRY(score),  ENTRY(compact),
                         ENTRY(compact_batch), ENTRY(frame_attn), ENTRY(rows), ENTRY(budget), ENTRY(segment_budgets),
                         ENTRY(past_frames), ENTRY(prunable_span), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// What this file was built against, for the loader to compare: it reads torch's tensors through inlined accessors
// and calls the library through the header's signatures, and neither is checked anywhere else.
PyMODINIT_FUNC PyInit__marshal() {
  PyObject* m = PyModule_Create(&module);
  if (m && (PyModule_AddStringConstant(m, "torch_version", PC_TORCH_VERSION) < 0 ||
            PyModule_AddIntConstant(m, "pc_version", PC_VERSION) < 0))
    Py_CLEAR(m);
  return m;
}
