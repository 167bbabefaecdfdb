// The Python wrappers of the short calls (binding.py), in native code: tensors are checked, outputs
// and workspaces allocated and the C entry point called on the current stream.  On prompts and
// batches that the GPU finishes in a few microseconds the interpreter's share of a call -- some 25
// attribute reads, three allocations, a stream object and the conversion of 15 to 25 arguments, 11
// of 17 us for a mask with gather -- is what bounds the loop; here it is about 3 us.
// Every function takes its arguments by position, None where an optional one is absent, and returns
// the outputs, or the library's status as an int when it is not 0.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <string>

#include "kvzap.h"

namespace {

using at::ScalarType;
using at::Tensor;
constexpr ScalarType BF16 = at::kBFloat16, F32 = at::kFloat, I32 = at::kInt, I64 = at::kLong;

const char* dtype_name(ScalarType t) {
  switch (t) {
    case at::kBFloat16: return "torch.bfloat16";
    case at::kFloat: return "torch.float32";
    case at::kInt: return "torch.int32";
    case at::kLong: return "torch.int64";
    case at::kByte: return "torch.uint8";
    case at::kHalf: return "torch.float16";
    case at::kDouble: return "torch.float64";
    default: return c10::toString(t);
  }
}

[[noreturn]] void fail(PyObject* type, const std::string& message) {
  PyErr_SetString(type, message.c_str());
  throw python_error();
}
void require(bool ok, const char* message) {
  if (!ok) fail(PyExc_ValueError, message);
}

Tensor tensor(PyObject* o, const char* name) {
  if (o == Py_None) fail(PyExc_ValueError, std::string(name) + " is required");
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, std::string(name) + " must be a tensor");
  return THPVariable_Unpack(o);
}
void check(const Tensor& t, ScalarType dtype, const char* name) {
  if (!t.is_cuda()) fail(PyExc_ValueError, std::string(name) + " must be a device tensor");
  if (t.scalar_type() != dtype)
    fail(PyExc_ValueError, std::string(name) + " must be " + dtype_name(dtype) + ", got " + dtype_name(t.scalar_type()));
  if (!t.is_contiguous()) fail(PyExc_ValueError, std::string(name) + " must be contiguous");
}
Tensor in(PyObject* o, ScalarType dtype, const char* name) {
  Tensor t = tensor(o, name);
  check(t, dtype, name);
  return t;
}
Tensor maybe(PyObject* o, ScalarType dtype, const char* name) {       // undefined if None
  return o == Py_None ? Tensor() : in(o, dtype, name);
}
void* ptr(const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
// nullptr for a tensor without elements' worth of rows, which the library takes for "none"
void* rows_ptr(const Tensor& t) { return t.size(0) > 0 ? t.data_ptr() : nullptr; }

void dims(const Tensor& t, int64_t n, const char* name) {
  if (t.dim() != n) fail(PyExc_ValueError, std::string(name) + " must have " + std::to_string(n) + " dimensions");
}
Tensor alloc(at::IntArrayRef shape, ScalarType dtype, const Tensor& like) {
  return at::empty(shape, at::TensorOptions().dtype(dtype).device(like.device()));
}

long long integer(PyObject* o) {                                       // int(o), as ctypes passes it on
  PyObject* i = PyNumber_Long(o);
  if (!i) throw python_error();
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(i);
  Py_DECREF(i);
  if (PyErr_Occurred()) throw python_error();
  return (long long)v;
}
// a number that is compared with a size: 16.0 is one, 16.5 is not
long long whole(PyObject* o, const char* message) {
  const long long v = integer(o);
  if (PyLong_CheckExact(o)) return v;
  PyObject* i = PyLong_FromLongLong(v);
  const int same = i ? PyObject_RichCompareBool(o, i, Py_EQ) : -1;
  Py_XDECREF(i);
  if (same < 0) throw python_error();
  require(same == 1, message);
  return v;
}
long long size_of(PyObject* o) {                                       // of an allocation: no float
  PyObject* i = PyNumber_Index(o);
  if (!i) throw python_error();
  const long long v = PyLong_AsLongLong(i);
  Py_DECREF(i);
  if (PyErr_Occurred()) throw python_error();
  return v;
}
double real(PyObject* o) {
  PyObject* f = PyNumber_Float(o);
  if (!f) throw python_error();
  const double v = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw python_error();
  return v != 0;
}

// None: the current stream of the current device; otherwise the handle as an int
void* stream_of(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  return reinterpret_cast<void*>((uintptr_t)integer(o));
}

// The caller's workspace, or one from the caching allocator (on the current stream: the wrappers
// pass one along with any other stream), as plain memory: nobody sees it, and a tensor around it costs more
// than it does (linear scorer, mask and gather of 1024 tokens, which the host bounds: 11.5 -> 11.1 us a pass).
struct Workspace {
  Tensor given;
  c10::DataPtr own;
  void* at = nullptr;
  size_t bytes = 0;
  Workspace(PyObject* o, size_t need, const Tensor& like) {
    if (o != Py_None) {
      given = tensor(o, "workspace");
      at = ptr(given);
      bytes = given.numel() * given.element_size();
    } else if (need > 0) {
      c10::DeviceGuard guard(like.device());
      own = c10::hip::HIPCachingAllocator::get()->allocate(need);
      at = own.get();
      bytes = need;
    }
  }
};

template <class F>
int call(F&& f) {                       // a launch may wait for room in the queue: without the GIL
  PyThreadState* save = PyEval_SaveThread();
  const int rc = f();
  PyEval_RestoreThread(save);
  return rc;
}

PyObject* none() { Py_RETURN_NONE; }
PyObject* status(int rc) { return PyLong_FromLong(rc); }
PyObject* give(const Tensor& t) { return THPVariable_Wrap(t); }
template <class... T>
PyObject* give_all(const T&... t) {
  PyObject* out = PyTuple_New(sizeof...(T));
  if (!out) throw python_error();
  Py_ssize_t i = 0;
  (PyTuple_SET_ITEM(out, i++, THPVariable_Wrap(t)), ...);
  return out;
}

#define KVZAP_FUNCTION(name, count)                                                       \
  PyObject* name##_body(PyObject* const* a);                                              \
  PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) {                           \
    HANDLE_TH_ERRORS                                                                      \
    if (n != (count)) fail(PyExc_TypeError, #name " takes " #count " arguments");  \
    return name##_body(a);                                                                \
    END_HANDLE_TH_ERRORS                                                                  \
  }                                                                                       \
  PyObject* name##_body(PyObject* const* a)

// hidden, W1, b1, W2, b2, scores, workspace, stream
KVZAP_FUNCTION(score, 8) {
  const Tensor hidden = in(a[0], BF16, "hidden"), W1 = in(a[1], BF16, "W1"), b1 = maybe(a[2], BF16, "b1"),
               W2 = maybe(a[3], BF16, "W2"), b2 = maybe(a[4], BF16, "b2");
  dims(hidden, 3, "hidden");
  const int64_t B = hidden.size(0), T = hidden.size(1), Dh = hidden.size(2);
  int64_t M = 0, H;
  if (W2.defined()) {
    require(W1.dim() == 2 && W2.dim() == 2 && W1.size(1) == Dh && W2.size(1) == W1.size(0), "W1 must be [M,Dh] and W2 [H,M]");
    M = W1.size(0);
    H = W2.size(0);
    require((!b1.defined() || (b1.dim() == 1 && b1.size(0) == M)) && (!b2.defined() || (b2.dim() == 1 && b2.size(0) == H)),
            "b1 must be [M] and b2 [H]");
  } else {
    require(W1.dim() == 2 && W1.size(1) == Dh && (!b1.defined() || (b1.dim() == 1 && b1.size(0) == W1.size(0))),
            "W1 must be [H,Dh] and b1 [H]");
    H = W1.size(0);
  }
  Tensor scores = maybe(a[5], F32, "scores");
  if (!scores.defined()) scores = alloc({B, H, T}, F32, hidden);
  require(scores.sizes() == at::IntArrayRef({B, H, T}), "scores must be [B,H,T]");
  const Workspace ws(a[6], kvzap_workspace_bytes(KVZAP_CALL_SCORE, B, T, Dh, M, H), hidden);
  void* stream = stream_of(a[7]);
  const int rc = call([&] {
    return kvzap_score(ptr(hidden), ptr(W1), ptr(b1), ptr(W2), ptr(b2), (float*)ptr(scores), B, T, Dh, M, H, ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give(scores);
}

// hidden, W1_prepared, b1, W2, b2, scores, workspace, stream
KVZAP_FUNCTION(score_prepared, 8) {
  const Tensor hidden = in(a[0], BF16, "hidden"), W1 = in(a[1], at::kByte, "W1_prepared"), b1 = maybe(a[2], BF16, "b1"),
               W2 = in(a[3], BF16, "W2"), b2 = maybe(a[4], BF16, "b2");
  dims(hidden, 3, "hidden");
  dims(W2, 2, "W2");
  const int64_t B = hidden.size(0), T = hidden.size(1), Dh = hidden.size(2), H = W2.size(0), M = W2.size(1);
  require(W1.numel() >= M * Dh * 2, "W1_prepared is smaller than M*Dh bf16 values");
  Tensor scores = maybe(a[5], F32, "scores");
  if (!scores.defined()) scores = alloc({B, H, T}, F32, hidden);
  require(scores.sizes() == at::IntArrayRef({B, H, T}), "scores must be [B,H,T]");
  const Workspace ws(a[6], kvzap_workspace_bytes(KVZAP_CALL_SCORE_PREPARED, B, T, Dh, M, H), hidden);
  void* stream = stream_of(a[7]);
  const int rc = call([&] {
    return kvzap_score_prepared_ws(ptr(hidden), ptr(W1), ptr(b1), ptr(W2), ptr(b2), (float*)ptr(scores), B, T, Dh, M, H, ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give(scores);
}

// x, W1_prepared, gain, eps, b1, W2, b2, want_normed, scores, rstd, normed, workspace, stream
KVZAP_FUNCTION(score_rmsnorm, 13) {
  const Tensor x = in(a[0], BF16, "x"), gain = in(a[2], BF16, "gain"), b1 = maybe(a[4], BF16, "b1"), W2 = in(a[5], BF16, "W2"),
               b2 = maybe(a[6], BF16, "b2"), W1 = tensor(a[1], "W1_prepared");
  dims(x, 3, "x");
  dims(W2, 2, "W2");
  const int64_t B = x.size(0), T = x.size(1), Dh = x.size(2), H = W2.size(0), M = W2.size(1);
  require(W1.scalar_type() == at::kByte && W1.numel() >= M * Dh * 2, "W1_prepared must come from kvzap_prepare_scorer_rmsnorm");
  require(gain.dim() == 1 && gain.size(0) == Dh, "gain must be [Dh]");
  const float eps = (float)real(a[3]);
  Tensor scores = maybe(a[8], F32, "scores"), rstd = maybe(a[9], F32, "rstd"), normed = maybe(a[10], BF16, "normed");
  if (!scores.defined()) scores = alloc({B, H, T}, F32, x);
  if (!rstd.defined()) rstd = alloc({B, T}, F32, x);
  if (!normed.defined() && truth(a[7])) normed = alloc({B, T, Dh}, BF16, x);
  require(scores.sizes() == at::IntArrayRef({B, H, T}) && rstd.sizes() == at::IntArrayRef({B, T}) &&
              (!normed.defined() || normed.sizes() == x.sizes()), "scores must be [B,H,T], rstd [B,T], normed like x");
  const Workspace ws(a[11], kvzap_workspace_bytes(KVZAP_CALL_SCORE_PREPARED, B, T, Dh, M, H), x);
  void* stream = stream_of(a[12]);
  const int rc = call([&] {
    return kvzap_score_rmsnorm_ws(ptr(x), ptr(W1), ptr(gain), eps, ptr(b1), ptr(W2), ptr(b2), (float*)ptr(scores), (float*)ptr(rstd),
                                  ptr(normed), B, T, Dh, M, H, ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give_all(scores, rstd, normed);
}

// what the three mask calls share: the packed index list, the lengths and the offsets
struct Lists {
  Tensor idx, lengths, offsets;
  Lists(PyObject* i, PyObject* l, PyObject* o, int64_t B, int64_t H, int64_t T, const Tensor& like, bool checked) {
    auto get = [&](PyObject* p, at::IntArrayRef shape, ScalarType dtype, const char* name) {
      if (p == Py_None) return alloc(shape, dtype, like);
      return checked ? in(p, dtype, name) : tensor(p, name);
    };
    idx = get(i, {B * H * T}, I32, "keep_idx");
    lengths = get(l, {B, H}, I32, "lengths");
    offsets = get(o, {B * H + 1}, I64, "offsets");
    if (checked)
      require(idx.numel() >= B * H * T && lengths.numel() == B * H && offsets.numel() == B * H + 1, "output buffers have the wrong size");
  }
};

// scores, tau, window, seq_lens, keep_idx, lengths, offsets, workspace, stream
KVZAP_FUNCTION(mask, 9) {
  const Tensor scores = in(a[0], F32, "scores"), seq = maybe(a[3], I32, "seq_lens");
  dims(scores, 3, "scores");
  const int64_t B = scores.size(0), H = scores.size(1), T = scores.size(2);
  const float tau = (float)real(a[1]);
  const int window = (int)integer(a[2]);
  const Lists out(a[4], a[5], a[6], B, H, T, scores, true);
  const Workspace ws(a[7], kvzap_workspace_bytes(KVZAP_CALL_MASK, B, T, 0, 0, H), scores);
  void* stream = stream_of(a[8]);
  const int rc = call([&] {
    return kvzap_mask((const float*)ptr(scores), tau, window, (const int32_t*)ptr(seq), B, H, T, (int32_t*)ptr(out.idx),
                      (int32_t*)ptr(out.lengths), (int64_t*)ptr(out.offsets), ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give_all(out.idx, out.lengths, out.offsets);
}

// scores, tau, window, seq_lens, keep_idx, lengths, offsets, workspace, stream
KVZAP_FUNCTION(mask_per_head, 9) {
  const Tensor scores = in(a[0], F32, "scores"), tau = in(a[1], F32, "tau"), seq = maybe(a[3], I32, "seq_lens");
  dims(scores, 3, "scores");
  const int64_t B = scores.size(0), H = scores.size(1), T = scores.size(2);
  require(tau.numel() == B * H, "tau must have B*H entries");
  const int window = (int)integer(a[2]);
  const Lists out(a[4], a[5], a[6], B, H, T, scores, false);
  const Workspace ws(a[7], kvzap_workspace_bytes(KVZAP_CALL_MASK, B, T, 0, 0, H), scores);
  void* stream = stream_of(a[8]);
  const int rc = call([&] {
    return kvzap_mask_per_head((const float*)ptr(scores), (const float*)ptr(tau), window, (const int32_t*)ptr(seq), B, H, T,
                               (int32_t*)ptr(out.idx), (int32_t*)ptr(out.lengths), (int64_t*)ptr(out.offsets), ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give_all(out.idx, out.lengths, out.offsets);
}

// scores, tau, window, K, V, seq_lens, keep_idx, lengths, offsets, K_out, V_out, cap_rows, workspace, stream
KVZAP_FUNCTION(mask_compact, 14) {
  const Tensor scores = in(a[0], F32, "scores"), K = in(a[3], BF16, "K"), V = in(a[4], BF16, "V"), seq = maybe(a[5], I32, "seq_lens");
  dims(scores, 3, "scores");
  const int64_t B = scores.size(0), H = scores.size(1), T = scores.size(2);
  require(K.dim() == 4 && K.size(0) == B && K.size(1) == H && K.size(2) == T && K.sizes() == V.sizes(), "K and V must be [B,H,T,D]");
  const int64_t D = K.size(3);
  const float tau = (float)real(a[1]);
  const int window = (int)integer(a[2]);
  const Lists out(a[6], a[7], a[8], B, H, T, scores, true);
  Tensor Ko = maybe(a[9], BF16, "K_out"), Vo = maybe(a[10], BF16, "V_out");
  const int64_t cap = a[11] != Py_None ? (Ko.defined() && Vo.defined() ? integer(a[11]) : size_of(a[11])) : Ko.defined() ? (dims(Ko, 2, "K_out"), Ko.size(0)) : B * H * T;
  if (!Ko.defined()) Ko = alloc({cap, D}, BF16, scores);
  if (!Vo.defined()) Vo = alloc({cap, D}, BF16, scores);
  require(Ko.dim() == 2 && Vo.dim() == 2 && Ko.size(0) >= cap && Vo.size(0) >= cap && Ko.size(1) == D && Vo.size(1) == D,
          "K_out and V_out must be [>= cap_rows, D]");
  const Workspace ws(a[12], std::max<size_t>(kvzap_workspace_bytes(KVZAP_CALL_MASK_COMPACT, B, T, 0, 0, H), 256), scores);
  void* stream = stream_of(a[13]);
  const int rc = call([&] {
    return kvzap_mask_compact((const float*)ptr(scores), tau, window, (const int32_t*)ptr(seq), ptr(K), ptr(V), (int32_t*)ptr(out.idx),
                              (int32_t*)ptr(out.lengths), (int64_t*)ptr(out.offsets), ptr(Ko), ptr(Vo), cap, B, H, T, D, ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give_all(out.idx, out.lengths, out.offsets, Ko, Vo);
}

// K, V, keep_idx, lengths, offsets, K_out, V_out, cap_rows, stream
KVZAP_FUNCTION(compact, 9) {
  const Tensor K = in(a[0], BF16, "K"), V = in(a[1], BF16, "V"), idx = in(a[2], I32, "keep_idx"), len = in(a[3], I32, "lengths"),
               off = in(a[4], I64, "offsets");
  dims(K, 4, "K");
  const int64_t B = K.size(0), H = K.size(1), T = K.size(2), D = K.size(3);
  require(V.sizes() == K.sizes(), "K and V must have the same shape");
  Tensor Ko = maybe(a[5], BF16, "K_out"), Vo = maybe(a[6], BF16, "V_out");
  const int64_t cap = a[7] != Py_None ? (Ko.defined() && Vo.defined() ? integer(a[7]) : size_of(a[7])) : Ko.defined() ? (dims(Ko, 2, "K_out"), Ko.size(0)) : B * H * T;
  if (!Ko.defined()) Ko = alloc({cap, D}, BF16, K);
  if (!Vo.defined()) Vo = alloc({cap, D}, BF16, K);
  require(Ko.dim() == 2 && Vo.dim() >= 1 && Ko.size(0) >= cap && Vo.size(0) >= cap && Ko.size(1) == D, "K_out / V_out smaller than cap_rows");
  void* stream = stream_of(a[8]);
  const int rc = call([&] {
    return kvzap_compact(ptr(K), ptr(V), (const int32_t*)ptr(idx), (const int32_t*)ptr(len), (const int64_t*)ptr(off), ptr(Ko), ptr(Vo),
                         cap, B, H, T, D, stream);
  });
  return rc ? status(rc) : give_all(Ko, Vo);
}

// K, V, keep_idx, lengths, offsets, block_table, page_rows, K_pool, V_pool, stream
KVZAP_FUNCTION(compact_paged, 10) {
  const Tensor K = in(a[0], BF16, "K"), V = in(a[1], BF16, "V"), Kp = in(a[7], BF16, "K_pool"), Vp = in(a[8], BF16, "V_pool"),
               idx = in(a[2], I32, "keep_idx"), len = in(a[3], I32, "lengths"), off = in(a[4], I64, "offsets"),
               table = in(a[5], I32, "block_table");
  dims(K, 4, "K");
  const int64_t B = K.size(0), H = K.size(1), T = K.size(2), D = K.size(3);
  const int64_t P = whole(a[6], "pools must be [num_pages, page_rows, D]");
  require(V.sizes() == K.sizes() && Kp.sizes() == Vp.sizes(), "K/V and the two pools must have matching shapes");
  require(Kp.dim() == 3 && Kp.size(1) == P && Kp.size(2) == D, "pools must be [num_pages, page_rows, D]");
  require(table.dim() == 2 && table.size(0) == B * H, "block_table must be [B*H, max_pages]");
  void* stream = stream_of(a[9]);
  const int rc = call([&] {
    return kvzap_compact_paged(ptr(K), ptr(V), (const int32_t*)ptr(idx), (const int32_t*)ptr(len), (const int64_t*)ptr(off),
                               (const int32_t*)ptr(table), table.size(1), P, rows_ptr(Kp), rows_ptr(Vp), Kp.size(0), B, H, T, D, stream);
  });
  return rc ? status(rc) : none();
}

// lengths, page_rows, free_pages, max_pages, reserve_rows, block_table, result, workspace, stream
KVZAP_FUNCTION(assign_pages, 9) {
  const Tensor len = in(a[0], I32, "lengths"), free_pages = in(a[2], I32, "free_pages");
  dims(len, 2, "lengths");
  const int64_t B = len.size(0), H = len.size(1);
  const int64_t max_pages = a[5] == Py_None ? size_of(a[3]) : whole(a[3], "block_table must be [B*H, max_pages]");
  const int page_rows = (int)integer(a[1]), reserve = (int)integer(a[4]);
  Tensor table = maybe(a[5], I32, "block_table"), result = maybe(a[6], I32, "result");
  if (!table.defined()) table = alloc({B * H, max_pages}, I32, len);
  require(table.sizes() == at::IntArrayRef({B * H, max_pages}), "block_table must be [B*H, max_pages]");
  if (!result.defined()) result = alloc({4}, I32, len);
  const Workspace ws(a[7], kvzap_workspace_bytes(KVZAP_CALL_ASSIGN_PAGES, B, 1, 0, 0, H), len);
  void* stream = stream_of(a[8]);
  const int64_t n_free = free_pages.numel();
  const int rc = call([&] {
    return kvzap_assign_pages((const int32_t*)ptr(len), B, H, page_rows, reserve, n_free ? (const int32_t*)ptr(free_pages) : nullptr, n_free,
                              (int32_t*)ptr(table), max_pages, (int32_t*)ptr(result), ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give_all(table, result);
}

// scores, window, k, per_layer, seq_lens, tau_out, workspace, stream
KVZAP_FUNCTION(topk_threshold, 8) {
  const Tensor scores = in(a[0], F32, "scores"), seq = maybe(a[4], I32, "seq_lens");
  dims(scores, 3, "scores");
  const int64_t B = scores.size(0), H = scores.size(1), T = scores.size(2);
  const int window = (int)integer(a[1]), per_layer = truth(a[3]);
  const int64_t k = integer(a[2]);
  Tensor tau = maybe(a[5], F32, "tau_out");
  if (!tau.defined()) tau = alloc({B, H}, F32, scores);
  const Workspace ws(a[6], kvzap_workspace_bytes(KVZAP_CALL_TOPK_THRESHOLD, B, T, 0, per_layer, H), scores);
  void* stream = stream_of(a[7]);
  const int rc = call([&] {
    return kvzap_topk_threshold((const float*)ptr(scores), window, (const int32_t*)ptr(seq), k, per_layer, B, H, T, (float*)ptr(tau),
                                ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give(tau);
}

// The decode state's buffers are the library's own (DecodeState, PagedDecodeState) and not checked.
struct Step {
  Tensor hidden, W1, b1, W2, b2, k, v;
  int64_t B, Dh, M;
  Step(PyObject* const* a, int64_t state_B, int64_t H, int64_t D)
      : hidden(in(a[0], BF16, "hidden_new")), W1(in(a[1], BF16, "W1")), b1(maybe(a[2], BF16, "b1")), W2(maybe(a[3], BF16, "W2")),
        b2(maybe(a[4], BF16, "b2")), k(in(a[5], BF16, "k_new")), v(in(a[6], BF16, "v_new")) {
    dims(hidden, 2, "hidden_new");
    B = hidden.size(0);
    Dh = hidden.size(1);
    M = W2.defined() ? W1.size(0) : 0;
    require(k.sizes() == at::IntArrayRef({B, H, D}) && k.sizes() == v.sizes() && B == state_B, "k_new / v_new must be [B,H,D] matching the state");
  }
};

// hidden_new, W1, b1, W2, b2, k_new, v_new | B, H, D, window, K_prefix, V_prefix, prefix_pos, slab_offsets,
// slab_capacity, K_ring, V_ring, score_ring, lengths, seq_pos, error_flag | tau, workspace, stream
KVZAP_FUNCTION(decode_evict, 25) {
  const int64_t H = integer(a[8]), D = integer(a[9]), window = integer(a[10]);
  const Step s(a, integer(a[7]), H, D);
  Tensor st[11];
  for (int i = 0; i < 11; ++i) st[i] = tensor(a[11 + i], "state");
  const float tau = (float)real(a[22]);
  const Workspace ws(a[23], kvzap_workspace_bytes(KVZAP_CALL_DECODE_EVICT, s.B, 1, s.Dh, s.M, H), s.hidden);
  void* stream = stream_of(a[24]);
  const bool ring = window > 0;
  return status(call([&] {
    return kvzap_decode_evict(ptr(s.hidden), ptr(s.W1), ptr(s.b1), ptr(s.W2), ptr(s.b2), s.Dh, s.M, ptr(s.k), ptr(s.v), ptr(st[0]), ptr(st[1]),
                              (int32_t*)ptr(st[2]), (const int64_t*)ptr(st[3]), (const int32_t*)ptr(st[4]), ring ? ptr(st[5]) : nullptr,
                              ring ? ptr(st[6]) : nullptr, ring ? (float*)ptr(st[7]) : nullptr, (int32_t*)ptr(st[8]), (int32_t*)ptr(st[9]), tau,
                              window, s.B, H, D, (int32_t*)ptr(st[10]), ws.at, ws.bytes, stream);
  }));
}

// hidden_new, W1, b1, W2, b2, k_new, v_new | B, H, D, window, K_pool, V_pool, pos_pool, block_table, K_ring, V_ring,
// score_ring, lengths, seq_pos, error_flag | num_pages, max_pages, page_rows, tau, workspace, stream
KVZAP_FUNCTION(decode_evict_paged, 27) {
  const int64_t H = integer(a[8]), D = integer(a[9]), window = integer(a[10]);
  const Step s(a, integer(a[7]), H, D);
  Tensor st[10];
  for (int i = 0; i < 10; ++i) st[i] = tensor(a[11 + i], "state");
  const int num_pages = (int)integer(a[21]), max_pages = (int)integer(a[22]), page_rows = (int)integer(a[23]);
  const float tau = (float)real(a[24]);
  const Workspace ws(a[25], kvzap_workspace_bytes(KVZAP_CALL_DECODE_EVICT, s.B, 1, s.Dh, s.M, H), s.hidden);
  void* stream = stream_of(a[26]);
  const bool ring = window > 0;
  return status(call([&] {
    return kvzap_decode_evict_paged(ptr(s.hidden), ptr(s.W1), ptr(s.b1), ptr(s.W2), ptr(s.b2), s.Dh, s.M, ptr(s.k), ptr(s.v), ptr(st[0]),
                                    ptr(st[1]), (int32_t*)ptr(st[2]), num_pages, (const int32_t*)ptr(st[3]), max_pages, page_rows,
                                    ring ? ptr(st[4]) : nullptr, ring ? ptr(st[5]) : nullptr, ring ? (float*)ptr(st[6]) : nullptr,
                                    (int32_t*)ptr(st[7]), (int32_t*)ptr(st[8]), tau, window, s.B, H, D, (int32_t*)ptr(st[9]), ws.at,
                                    ws.bytes, stream);
  }));
}

int64_t ring_size(PyObject* o) {                                       // not positive: no ring
  if (PyLong_CheckExact(o) || real(o) > 0.0) return whole(o, "K_ring and V_ring must be [B,H,window,D]");
  return integer(o);
}

// q, K_rows, V_rows, row_offsets, lengths, K_ring, V_ring, seq_pos, window, max_rows, scale, out, workspace, stream
KVZAP_FUNCTION(attend_decode, 14) {
  const Tensor q = in(a[0], BF16, "q"), K = in(a[1], BF16, "K_rows"), V = in(a[2], BF16, "V_rows"), off = in(a[3], I64, "row_offsets"),
               len = in(a[4], I32, "lengths");
  dims(q, 3, "q");
  const int64_t B = q.size(0), HQ = q.size(1), D = q.size(2), window = ring_size(a[8]), max_rows = integer(a[9]);
  require(len.dim() == 2 && len.size(0) == B, "lengths must be [B,H]");
  const int64_t H = len.size(1);
  require(off.numel() == B * H, "row_offsets must have B*H entries");
  require(K.dim() == 2 && K.size(1) == D && K.sizes() == V.sizes(), "K_rows and V_rows must both be [total_rows, D]");
  Tensor Kr, Vr, pos;
  if (window > 0) {
    Kr = in(a[5], BF16, "K_ring");
    Vr = in(a[6], BF16, "V_ring");
    pos = in(a[7], I32, "seq_pos");
    require(Kr.sizes() == at::IntArrayRef({B, H, window, D}) && Kr.sizes() == Vr.sizes(), "K_ring and V_ring must be [B,H,window,D]");
    require(pos.numel() == B, "seq_pos must have B entries");
  }
  const float scale = (float)real(a[10]);
  Tensor out = maybe(a[11], BF16, "out");
  if (!out.defined()) out = alloc({B, HQ, D}, BF16, q);
  require(out.sizes() == q.sizes(), "out must be [B,HQ,D]");
  const Workspace ws(a[12], kvzap_workspace_bytes(KVZAP_CALL_ATTEND_DECODE, B, max_rows, HQ, window, H), q);
  void* stream = stream_of(a[13]);
  const int rc = call([&] {
    return kvzap_attend_decode(ptr(q), rows_ptr(K), rows_ptr(V), K.size(0), (const int64_t*)ptr(off), (const int32_t*)ptr(len), ptr(Kr), ptr(Vr),
                               (const int32_t*)ptr(pos), window, max_rows, scale, ptr(out), B, H, HQ, D, ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give(out);
}

// q, K_pool, V_pool, block_table, page_rows, lengths, K_ring, V_ring, seq_pos, window, max_rows, scale, out, workspace, stream
KVZAP_FUNCTION(attend_decode_paged, 15) {
  const Tensor q = in(a[0], BF16, "q"), K = in(a[1], BF16, "K_pool"), V = in(a[2], BF16, "V_pool"), table = in(a[3], I32, "block_table"),
               len = in(a[5], I32, "lengths");
  dims(q, 3, "q");
  const int64_t B = q.size(0), HQ = q.size(1), D = q.size(2), window = ring_size(a[9]), max_rows = integer(a[10]);
  const int64_t P = whole(a[4], "pools must both be [num_pages, page_rows, D]");
  require(len.dim() == 2 && len.size(0) == B, "lengths must be [B,H]");
  const int64_t H = len.size(1);
  require(K.dim() == 3 && K.size(1) == P && K.size(2) == D && K.sizes() == V.sizes(), "pools must both be [num_pages, page_rows, D]");
  require(table.dim() == 2 && table.size(0) == B * H, "block_table must be [B*H, max_pages]");
  Tensor Kr, Vr, pos;
  if (window > 0) {
    Kr = in(a[6], BF16, "K_ring");
    Vr = in(a[7], BF16, "V_ring");
    pos = in(a[8], I32, "seq_pos");
    require(Kr.sizes() == at::IntArrayRef({B, H, window, D}) && Kr.sizes() == Vr.sizes(), "K_ring and V_ring must be [B,H,window,D]");
  }
  const float scale = (float)real(a[11]);
  Tensor out = maybe(a[12], BF16, "out");
  if (!out.defined()) out = alloc({B, HQ, D}, BF16, q);
  const Workspace ws(a[13], kvzap_workspace_bytes(KVZAP_CALL_ATTEND_DECODE, B, max_rows, HQ, window, H), q);
  void* stream = stream_of(a[14]);
  const int rc = call([&] {
    return kvzap_attend_decode_paged(ptr(q), rows_ptr(K), rows_ptr(V), K.size(0), (const int32_t*)ptr(table), table.size(1), P,
                                     (const int32_t*)ptr(len), ptr(Kr), ptr(Vr), (const int32_t*)ptr(pos), window, max_rows, scale, ptr(out),
                                     B, H, HQ, D, ws.at, ws.bytes, stream);
  });
  return rc ? status(rc) : give(out);
}

#define KVZAP_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    KVZAP_METHOD(score), KVZAP_METHOD(score_prepared), KVZAP_METHOD(score_rmsnorm), KVZAP_METHOD(mask), KVZAP_METHOD(mask_per_head), KVZAP_METHOD(mask_compact),
    KVZAP_METHOD(compact), KVZAP_METHOD(compact_paged), KVZAP_METHOD(assign_pages), KVZAP_METHOD(topk_threshold),
    KVZAP_METHOD(decode_evict), KVZAP_METHOD(decode_evict_paged), KVZAP_METHOD(attend_decode), KVZAP_METHOD(attend_decode_paged),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kvzap_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kvzap_host() { return PyModule_Create(&module); }
