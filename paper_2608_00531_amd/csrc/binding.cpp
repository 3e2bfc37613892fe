// Python binding of the libcure calls that a decoding loop makes (the extension
// module _lib/_native). It checks and marshals arguments, allocates outputs as
// torch tensors and calls the C ABI on the tensors' current stream; cure.py holds
// the documented functions and calls these with positional arguments.
//
// Native because of what the calls cost next to their kernels. Per pass of calls
// in a row, marshalled in Python and here: cure_accept and cure_commit (10
// outputs) 35.1 and 16.9 us for 10 us of kernels, cure_margins and
// cure_repair_tree (12 outputs) 49.2 and 26.6 for 25, cure_margins_accept (13
// outputs) on 256 rows 34.3 and 20.1 for 15, a small cure_tree_attn 17.9 and 7.3.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "cure.h"

namespace {

PyObject* g_error = nullptr;      // cure.CureError
PyObject* g_host_i32 = nullptr;   // object -> C-contiguous numpy int32 array

// Thrown after a Python error has been set.
struct PyError {};

[[noreturn]] void fail(const std::string& what) {
  PyErr_SetString(g_error, what.c_str());
  throw PyError{};
}

void check(cure_status st, const char* what) {
  if (st != CURE_OK) fail(std::string(what) + " failed: " + cure_status_string(st));
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
    throw PyError{};
  }
  return THPVariable_Unpack(o);
}

at::Tensor gpu_tensor(PyObject* o) {
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda()) fail("tensor arguments must live on the GPU");
  return t;
}

// Integers and reals as ctypes takes them: anything with __index__, truncated
// to the C type; anything with __float__.
int32_t as_i32(PyObject* o) {
  if (PyFloat_Check(o)) {
    PyErr_SetString(PyExc_TypeError, "int expected instead of float instance");
    throw PyError{};
  }
  const unsigned long v = PyLong_AsUnsignedLongMask(o);
  if (v == (unsigned long)-1 && PyErr_Occurred()) throw PyError{};
  return (int32_t)(uint32_t)v;
}

float as_f32(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw PyError{};
  return (float)v;
}

bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw PyError{};
  return v != 0;
}

int32_t dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return CURE_F32;
  if (t.scalar_type() == at::kBFloat16) return CURE_BF16;
  PyObject* d = reinterpret_cast<PyObject*>(torch::getTHPDtype(t.scalar_type()));
  PyErr_Format(g_error, "unsupported dtype %S (float32 or bfloat16)", d);
  throw PyError{};
}

void* stream_of(const at::Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

at::Tensor empty(c10::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) {
  return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}

// Zero-filled device workspace, reused per (kind, device, stream) and grown when
// a call needs more; lives as long as the process. A graph captured on the stream
// holds its address, so a buffer that has become too small stays allocated, and
// each one is twice the last or more: those kept take less than the one in use.
// (Where twice the last does not fit on the GPU, what the call needs may.)
// The table is guarded by the GIL. A call holds `enqueue` while it enqueues its
// kernels: they pass data through the workspace, so another call's must not come
// between them on the stream.
struct Workspace {
  void* ptr;
  size_t bytes;
  std::mutex* enqueue;
};
enum Kind { kMargins, kAttn, kRepair };
Workspace workspace(Kind kind, const at::Tensor& like, void* stream, size_t bytes) {
  if (bytes == 0) return {nullptr, 0, nullptr};
  struct Slot {
    std::vector<at::Tensor> buffers;   // the last one is in use
    std::mutex enqueue;
  };
  static auto* kept = new std::map<std::tuple<int, int, void*>, Slot>;
  Slot& slot = (*kept)[{(int)kind, (int)like.device().index(), stream}];
  const size_t had = slot.buffers.empty() ? 0 : (size_t)slot.buffers.back().numel();
  if (had < bytes) {
    const auto zeros = [&](size_t n) {
      return at::zeros({(int64_t)n}, at::TensorOptions().dtype(at::kByte).device(like.device()));
    };
    at::Tensor grown;
    try {
      grown = zeros(std::max<size_t>({bytes, 2 * had, 256}));
    } catch (const c10::OutOfMemoryError&) {
      if (2 * had <= bytes) throw;
      grown = zeros(bytes);
    }
    slot.buffers.push_back(std::move(grown));
  }
  const at::Tensor& ws = slot.buffers.back();
  return {ws.data_ptr(), (size_t)ws.numel(), &slot.enqueue};
}
// The same for the scratch array inside the library that cure_margins_noalloc
// calls share.
std::mutex g_noalloc;

// The outputs of a call, in the order they are returned in.
struct Outputs {
  PyObject* dict = PyDict_New();
  Outputs() {
    if (!dict) throw PyError{};
  }
  ~Outputs() { Py_XDECREF(dict); }
  Outputs(const Outputs&) = delete;
  template <typename T>
  T* add(PyObject* key, at::Tensor t) {
    T* p = static_cast<T*>(t.data_ptr());
    PyObject* o = THPVariable_Wrap(std::move(t));
    if (!o) throw PyError{};
    const int bad = PyDict_SetItem(dict, key, o);
    Py_DECREF(o);
    if (bad) throw PyError{};
    return p;
  }
  PyObject* take() {
    PyObject* d = dict;
    dict = nullptr;
    return d;
  }
};

#define CURE_KEYS(X)                                                                     \
  X(top1_val) X(top1_idx) X(top2_val) X(top2_idx) X(lse) X(margin) X(ufp_pos) X(ufp_cnt) \
  X(acc_len) X(path) X(best) X(bonus) X(resync) X(parent) X(token) X(n_nodes)            \
  X(branch_cnt) X(new_ctx_len) X(emit) X(emit_cnt) X(replay_start) X(status)
#define X(name) PyObject* k_##name = nullptr;
CURE_KEYS(X)
#undef X

// Calls of the C ABI release the GIL, as a foreign call does. f touches no tensor
// and no Python object: its pointers are taken before (data_ptr() throws for a
// tensor without storage, as under vmap). `order`, if any, is held during the call;
// it is only ever waited for without the GIL.
template <typename F>
cure_status unlocked(F&& f, std::mutex* order = nullptr) {
  struct Released {
    PyThreadState* state = PyEval_SaveThread();
    ~Released() { PyEval_RestoreThread(state); }
  } released;
  std::unique_lock<std::mutex> held;
  if (order) held = std::unique_lock<std::mutex>(*order);
  return f();
}

void need_args(Py_ssize_t got, Py_ssize_t want) {
  if (got == want) return;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, got);
  throw PyError{};
}

// Logits as [batch, rows, vocab] with unit stride along the vocabulary and one
// row stride throughout; copied only when they are not.
at::Tensor logits_of(PyObject* o) {
  at::Tensor x = gpu_tensor(o);
  if (x.dim() == 2) x = x.unsqueeze(0);
  if (x.dim() != 3) {
    PyErr_SetString(PyExc_ValueError, "logits must be [batch, rows, vocab] or [rows, vocab]");
    throw PyError{};
  }
  if (x.stride(2) != 1 || x.stride(0) != x.size(1) * x.stride(1)) x = x.contiguous();
  return x;
}

const int32_t* i32_ptr(const at::Tensor& t) { return static_cast<const int32_t*>(t.data_ptr()); }

template <typename F>
PyObject* guarded(F&& f) {
  HANDLE_TH_ERRORS
  try {
    return f();
  } catch (const PyError&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

// margins(logits, chain_len, tau, repair_budget, branch_depth, gate, noalloc)
// margins(..., parent, token, root_tgt, n_nodes): with the acceptance walk
PyObject* py_margins(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    const bool accept = n == 11;
    need_args(n, accept ? 11 : 7);
    at::Tensor tree[4];
    if (accept)
      for (int i = 0; i < 4; ++i) tree[i] = gpu_tensor(args[7 + i]).contiguous();
    const at::Tensor x = logits_of(args[0]);
    const int32_t chain = as_i32(args[1]), budget = as_i32(args[3]), depth = as_i32(args[4]);
    const float tau = as_f32(args[2]);
    const bool gate = truth(args[5]), noalloc = truth(args[6]);
    const int32_t dtype = dtype_code(x);
    const int64_t batch = x.size(0), rows = x.size(1), vocab = x.size(2);
    Outputs out;
    float* v1 = out.add<float>(k_top1_val, empty({batch, rows}, at::kFloat, x));
    int32_t* i1 = out.add<int32_t>(k_top1_idx, empty({batch, rows}, at::kInt, x));
    float* v2 = out.add<float>(k_top2_val, empty({batch, rows}, at::kFloat, x));
    int32_t* i2 = out.add<int32_t>(k_top2_idx, empty({batch, rows}, at::kInt, x));
    float* lse = out.add<float>(k_lse, empty({batch, rows}, at::kFloat, x));
    float* margin = out.add<float>(k_margin, empty({batch, rows}, at::kFloat, x));
    int32_t *acc_len = nullptr, *path = nullptr, *best = nullptr, *bonus = nullptr, *resync = nullptr;
    if (accept) {
      acc_len = out.add<int32_t>(k_acc_len, empty({batch}, at::kInt, x));
      path = out.add<int32_t>(k_path, empty({batch, rows}, at::kInt, x));
      best = out.add<int32_t>(k_best, empty({batch}, at::kInt, x));
      bonus = out.add<int32_t>(k_bonus, empty({batch}, at::kInt, x));
      resync = out.add<int32_t>(k_resync, empty({batch}, at::kInt, x));
    }
    int32_t *pos = nullptr, *cnt = nullptr;
    if (gate) {
      pos = out.add<int32_t>(k_ufp_pos, empty({batch, chain}, at::kInt, x));
      cnt = out.add<int32_t>(k_ufp_cnt, empty({batch}, at::kInt, x));
    }
    void* s = stream_of(x);
    const int32_t b = (int32_t)batch, r = (int32_t)rows, v = (int32_t)vocab;
    const void* lp = x.data_ptr();
    const int32_t* tp[4] = {};           // parent, token, root_tgt, n_nodes
    if (accept)
      for (int i = 0; i < 4; ++i) tp[i] = i32_ptr(tree[i]);
    const int64_t ld = x.stride(1);
    if (noalloc) {
      check(unlocked([&] {
              return cure_margins_noalloc(lp, dtype, b, r, v, ld, v1, i1, v2, i2, lse, margin, chain, tau,
                                          budget, depth, pos, cnt, s);
            }, &g_noalloc), "cure_margins_noalloc");
      return out.take();
    }
    const Workspace ws = workspace(kMargins, x, s, cure_margins_workspace_size(b, r, v));
    if (accept)
      check(unlocked([&] {
              return cure_margins_accept(lp, dtype, b, r, v, ld, v1, i1, v2, i2, lse, margin, chain, tau,
                                         budget, depth, pos, cnt, tp[0], tp[1], tp[2], tp[3], acc_len, path,
                                         best, bonus, resync, ws.ptr, ws.bytes, s);
            }, ws.enqueue), "cure_margins_accept");
    else
      check(unlocked([&] {
              return cure_margins(lp, dtype, b, r, v, ld, v1, i1, v2, i2, lse, margin, chain, tau, budget,
                                  depth, pos, cnt, ws.ptr, ws.bytes, s);
            }, ws.enqueue), "cure_margins");
    return out.take();
  });
}

// Host copies of per-sequence sizes: lists of ints directly, anything else
// through numpy.
std::vector<int32_t> host_sizes(PyObject* o, int64_t batch) {
  std::vector<int32_t> v;
  if (PyList_CheckExact(o)) {
    const Py_ssize_t n = PyList_GET_SIZE(o);
    v.reserve(n);
    for (Py_ssize_t i = 0; i < n; ++i) {
      PyObject* e = PyList_GET_ITEM(o, i);
      int overflow = 0;
      const long x = PyLong_CheckExact(e) ? PyLong_AsLongAndOverflow(e, &overflow) : -1;
      if (!PyLong_CheckExact(e) || overflow || x != (int32_t)x) break;
      v.push_back((int32_t)x);
    }
    if ((Py_ssize_t)v.size() != n) v.clear();
    else if (v.size() >= (size_t)batch) return v;
  }
  PyObject* a = PyObject_CallOneArg(g_host_i32, o);
  if (!a) throw PyError{};
  Py_buffer buf;
  const int bad = PyObject_GetBuffer(a, &buf, PyBUF_C_CONTIGUOUS);
  Py_DECREF(a);
  if (bad) throw PyError{};
  const int32_t* p = static_cast<const int32_t*>(buf.buf);
  v.assign(p, p + buf.len / sizeof(int32_t));
  PyBuffer_Release(&buf);
  if (v.size() < (size_t)batch) fail("host sizes are shorter than the batch");
  return v;
}

// tree_attn(q, k, v, kv_off, ctx_len, n_nodes, parent, host_ctx_len, host_n_nodes, scale,
//           out_dtype, kv_split, flags, with_lse)
PyObject* py_tree_attn(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    need_args(n, 14);
    at::Tensor t[7];
    for (int i = 0; i < 7; ++i) t[i] = gpu_tensor(args[i]);
    for (const at::Tensor& x : t)
      if (!x.is_contiguous()) fail("tree attention arguments must be contiguous");
    const at::Tensor &q = t[0], &k = t[1], &v = t[2], &kv_off = t[3], &ctx = t[4], &nn = t[5], &par = t[6];
    if (kv_off.scalar_type() != at::kLong || ctx.scalar_type() != at::kInt || nn.scalar_type() != at::kInt ||
        par.scalar_type() != at::kInt)
      fail("kv_off must be int64; ctx_len, n_nodes and parent int32");
    if (q.dim() != 4 || k.dim() < 2) {
      PyErr_SetString(PyExc_ValueError, "q must be [batch, n_max, hq, d], k and v [rows, hkv, d]");
      throw PyError{};
    }
    const int64_t batch = q.size(0), n_max = q.size(1), hq = q.size(2), d = q.size(3), hkv = k.size(1);
    at::ScalarType out_type = q.scalar_type();
    if (args[10] != Py_None) {
      if (!THPDtype_Check(args[10])) {
        PyErr_SetString(PyExc_TypeError, "out_dtype must be a torch.dtype");
        throw PyError{};
      }
      out_type = reinterpret_cast<THPDtype*>(args[10])->scalar_type;
    }
    const float scale = as_f32(args[9]);
    const int32_t split = as_i32(args[11]);
    const uint32_t flags = (uint32_t)as_i32(args[12]);
    const bool with_lse = truth(args[13]);
    const std::vector<int32_t> hc = host_sizes(args[7], batch), hn = host_sizes(args[8], batch);
    at::Tensor o = empty({batch, n_max, hq, d}, out_type, q);
    at::Tensor lse = with_lse ? empty({batch, n_max, hq}, at::kFloat, q) : at::Tensor();
    at::Tensor status = empty({batch}, at::kInt, q);
    const int32_t dt = dtype_code(q), odt = dtype_code(o);
    void* s = stream_of(q);
    const Workspace ws = workspace(kAttn, q, s, cure_tree_attn_workspace_size(
        (int32_t)batch, (int32_t)hq, (int32_t)hkv, (int32_t)d, (int32_t)n_max, hc.data(), hn.data(), split));
    const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
    void* op = o.data_ptr();
    float* lsep = with_lse ? static_cast<float*>(lse.data_ptr()) : nullptr;
    const int64_t* offp = static_cast<const int64_t*>(kv_off.data_ptr());
    const int32_t *cp = i32_ptr(ctx), *np = i32_ptr(nn), *pp = i32_ptr(par);
    int32_t* stp = static_cast<int32_t*>(status.data_ptr());
    check(unlocked([&] {
            return cure_tree_attn(qp, kp, vp, op, lsep, dt, odt, (int32_t)batch, (int32_t)hq, (int32_t)hkv,
                                  (int32_t)d, scale, offp, cp, np, pp, (int32_t)n_max, hc.data(), hn.data(),
                                  split, flags, stp, ws.ptr, ws.bytes, s);
          }, ws.enqueue), "cure_tree_attn");
    PyObject* r = PyTuple_New(3);
    if (!r) throw PyError{};
    PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(o));
    if (with_lse) {
      PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(lse));
    } else {
      Py_INCREF(Py_None);
      PyTuple_SET_ITEM(r, 1, Py_None);
    }
    PyTuple_SET_ITEM(r, 2, THPVariable_Wrap(status));
    return r;
  });
}

// accept(parent, token, tgt, root_tgt, n_nodes, chain_len)
PyObject* py_accept(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    need_args(n, 6);
    at::Tensor t[5];
    for (int i = 0; i < 5; ++i) t[i] = gpu_tensor(args[i]);
    if (t[0].dim() != 2) {
      PyErr_SetString(PyExc_ValueError, "parent must be [batch, n_max]");
      throw PyError{};
    }
    const int64_t batch = t[0].size(0), n_max = t[0].size(1);
    for (at::Tensor& x : t) x = x.contiguous();
    const int32_t chain = as_i32(args[5]);
    Outputs out;
    int32_t* len = out.add<int32_t>(k_acc_len, empty({batch}, at::kInt, t[0]));
    int32_t* path = out.add<int32_t>(k_path, empty({batch, n_max}, at::kInt, t[0]));
    int32_t* best = out.add<int32_t>(k_best, empty({batch}, at::kInt, t[0]));
    int32_t* bonus = out.add<int32_t>(k_bonus, empty({batch}, at::kInt, t[0]));
    int32_t* resync = out.add<int32_t>(k_resync, empty({batch}, at::kInt, t[0]));
    void* s = stream_of(t[0]);
    const int32_t* p[5];
    for (int i = 0; i < 5; ++i) p[i] = i32_ptr(t[i]);
    check(unlocked([&] {
            return cure_accept(p[0], p[1], p[2], p[3], p[4], chain, (int32_t)batch, (int32_t)n_max, len, path,
                               best, bonus, resync, s);
          }), "cure_accept");
    return out.take();
  });
}

std::string shape_text(c10::IntArrayRef s) {
  std::string t = "(";
  for (size_t i = 0; i < s.size(); ++i) t += (i ? ", " : "") + std::to_string(s[i]);
  return t + (s.size() == 1 ? ",)" : ")");
}

// repair_tree(logits, margin, ufp_pos, ufp_cnt, chain_tok, repair_budget, branch_depth,
//             margin_scale, b_min, b_max, suffix, n_max)
PyObject* py_repair_tree(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    need_args(n, 12);
    const at::Tensor x = logits_of(args[0]);
    at::Tensor t[5];                     // margin, ufp_pos, ufp_cnt, chain_tok, suffix
    for (int i = 0; i < 4; ++i) t[i] = gpu_tensor(args[1 + i]);
    const bool has_suffix = args[10] != Py_None;
    if (has_suffix) t[4] = gpu_tensor(args[10]);
    const int64_t batch = x.size(0), rows = x.size(1), vocab = x.size(2);
    if (t[3].dim() < 1) {
      PyErr_SetString(PyExc_IndexError, "chain_tok must be [batch, chain_len]");
      throw PyError{};
    }
    const int64_t chain = t[3].size(-1);
    bool ints = true;
    for (int i = 1; i < 4 + has_suffix; ++i) ints = ints && t[i].scalar_type() == at::kInt;
    if (t[0].scalar_type() != at::kFloat || !ints)
      fail("margin must be float32; ufp_pos, ufp_cnt, chain_tok and suffix int32");
    const int32_t budget = as_i32(args[5]), depth = as_i32(args[6]);
    const float scale = as_f32(args[7]);
    const int32_t b_min = as_i32(args[8]), b_max = as_i32(args[9]);
    const auto want = [](const at::Tensor& a, c10::IntArrayRef s) {
      if (a.sizes() != s) fail("expected shape " + shape_text(s) + ", got " + shape_text(a.sizes()));
    };
    want(t[0], {batch, rows});
    want(t[1], {batch, chain});
    want(t[2], {batch});
    want(t[3], {batch, chain});
    if (has_suffix && depth > 1) want(t[4], {batch, chain, b_max, depth - 1});
    const bool use_suffix = has_suffix && depth != 1;
    for (int i = 0; i < 4 + use_suffix; ++i) t[i] = t[i].contiguous();
    const int64_t n_max = args[11] == Py_None ? chain + budget : as_i32(args[11]);
    Outputs out;
    int32_t* parent = out.add<int32_t>(k_parent, empty({batch, n_max}, at::kInt, x));
    int32_t* token = out.add<int32_t>(k_token, empty({batch, n_max}, at::kInt, x));
    int32_t* nodes = out.add<int32_t>(k_n_nodes, empty({batch}, at::kInt, x));
    int32_t* branches = out.add<int32_t>(k_branch_cnt, empty({batch, chain}, at::kInt, x));
    void* s = stream_of(x);
    const Workspace ws = workspace(kRepair, x, s, cure_repair_tree_workspace_size(
        (int32_t)batch, (int32_t)chain, (int32_t)vocab, budget, depth));
    const int32_t dtype = dtype_code(x);
    const void* lp = x.data_ptr();
    const int64_t ld = x.stride(1);
    const float* mp = static_cast<const float*>(t[0].data_ptr());
    const int32_t *pos = i32_ptr(t[1]), *cnt = i32_ptr(t[2]), *tok = i32_ptr(t[3]);
    const int32_t* suffix = use_suffix ? i32_ptr(t[4]) : nullptr;
    check(unlocked([&] {
            return cure_repair_tree(lp, dtype, (int32_t)batch, (int32_t)rows, (int32_t)vocab, ld, mp, pos, cnt,
                                    tok, (int32_t)chain, budget, depth, scale, b_min, b_max, suffix,
                                    (int32_t)n_max, parent, token, nodes, branches, ws.ptr, ws.bytes, s);
          }, ws.enqueue), "cure_repair_tree");
    return out.take();
  });
}

// commit(k, v, kv_off, ctx_len, n_nodes, path, acc_len, token, bonus, chain_len, layer_stride)
PyObject* py_commit(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    need_args(n, 11);
    at::Tensor t[9];                     // k, v, kv_off, ctx_len, n_nodes, path, acc_len, token, bonus
    for (int i = 0; i < 9; ++i) t[i] = gpu_tensor(args[i]);
    const at::Tensor &k = t[0], &v = t[1];
    if (k.sizes() != v.sizes() || k.scalar_type() != v.scalar_type() || (k.dim() != 3 && k.dim() != 4))
      fail("k and v must have the same shape [n_layers,] rows, hkv, d");
    bool ints = t[2].scalar_type() == at::kLong;
    for (int i = 3; i < 9; ++i) ints = ints && t[i].scalar_type() == at::kInt;
    if (!ints) fail("kv_off must be int64; the other index arrays int32");
    const int64_t layers = k.dim() == 3 ? 1 : k.size(0), hkv = k.size(-2), d = k.size(-1);
    for (const at::Tensor& x : {k, v})
      if (x.stride(-3) != hkv * d || x.stride(-2) != d || x.stride(-1) != 1)
        fail("each layer of k and v must be contiguous");
    int64_t stride = k.dim() == 3 ? 0 : k.stride(0);
    if (args[10] != Py_None) {
      stride = PyLong_AsLongLong(args[10]);
      if (stride == -1 && PyErr_Occurred()) throw PyError{};
    }
    if (k.dim() == 4 && (k.stride(0) != stride || v.stride(0) != stride))
      fail("layer_stride does not match the tensors' layer stride");
    if (t[5].dim() != 2) {
      PyErr_SetString(PyExc_ValueError, "path must be [batch, n_max]");
      throw PyError{};
    }
    const int64_t batch = t[5].size(0), n_max = t[5].size(1);
    const int32_t chain = as_i32(args[9]);
    Outputs out;
    int32_t* ctx = out.add<int32_t>(k_new_ctx_len, empty({batch}, at::kInt, k));
    int32_t* emit = out.add<int32_t>(k_emit, empty({batch, n_max + 1}, at::kInt, k));
    int32_t* cnt = out.add<int32_t>(k_emit_cnt, empty({batch}, at::kInt, k));
    int32_t* replay = out.add<int32_t>(k_replay_start, empty({batch}, at::kInt, k));
    int32_t* status = out.add<int32_t>(k_status, empty({batch}, at::kInt, k));
    for (int i = 2; i < 9; ++i) t[i] = t[i].contiguous();
    const int32_t dtype = dtype_code(k);
    void* s = stream_of(k);
    void *kp = k.data_ptr(), *vp = v.data_ptr();
    const int64_t* offp = static_cast<const int64_t*>(t[2].data_ptr());
    const int32_t* p[6];                 // ctx_len, n_nodes, path, acc_len, token, bonus
    for (int i = 0; i < 6; ++i) p[i] = i32_ptr(t[3 + i]);
    check(unlocked([&] {
            return cure_commit(kp, vp, dtype, (int32_t)layers, stride, (int32_t)hkv, (int32_t)d, (int32_t)batch,
                               offp, p[0], p[1], p[2], p[3], p[4], p[5], chain, (int32_t)n_max, ctx, emit, cnt,
                               replay, status, s);
          }), "cure_commit");
    return out.take();
  });
}

// setup(CureError, host_i32)
PyObject* py_setup(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    need_args(n, 2);
    Py_INCREF(args[0]);
    Py_XSETREF(g_error, args[0]);
    Py_INCREF(args[1]);
    Py_XSETREF(g_host_i32, args[1]);
    Py_RETURN_NONE;
  });
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(setup),       FAST(margins), FAST(tree_attn), FAST(accept),
                         FAST(repair_tree), FAST(commit),  {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
#define X(name) \
  if (!(k_##name = PyUnicode_InternFromString(#name))) return nullptr;
  CURE_KEYS(X)
#undef X
  return PyModule_Create(&module);
}
