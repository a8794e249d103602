// Native marshalling of the calls a decode step makes many times: the argument
// checks of the Python binding (device placement, dtype, contiguity, element
// counts) and the call into liboasis.so in one extension call.
//
// Each function takes the arguments of the binding's function of that name and
// returns the library's status, or None when it does not accept them exactly as
// they are (an argument of another type, a tensor subclass, a failed check, a
// null argument that some sizes allow): the binding's Python code then handles
// the call, so that every error and every unusual form stays there. Nothing is
// kept between calls. Measured on the host of an MI355X, the attention call's
// marshalling takes 6.2 us in Python and 0.4 us here, more than a launch.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <cstdint>
#include <initializer_list>

#include "oasis.h"

namespace {

decltype(&oasis_sparse_decode_attn) f_attn;
decltype(&oasis_score_blocks) f_score;
decltype(&oasis_select_topk) f_topk;
decltype(&oasis_score_select) f_score_select;
decltype(&oasis_stage_blocks) f_stage;

enum Kind { kBf16, kI32, kF32, kU8 };

bool dtype_is(at::ScalarType t, Kind k) {
  switch (k) {
    case kBf16: return t == at::kBFloat16 || t == at::kUInt16 || t == at::kShort;  // bf16 bits in any 16-bit dtype
    case kI32: return t == at::kInt;
    case kF32: return t == at::kFloat;
    default: return t == at::kByte;
  }
}

// Product of counts; -1, which no tensor matches, with a negative factor or past 63 bits.
int64_t count(std::initializer_list<int64_t> factors) {
  int64_t n = 1;
  bool bad = false;
  for (const int64_t f : factors) bad |= f < 0 || __builtin_mul_overflow(n, f, &n);
  return bad ? -1 : n;
}

// The data of a plain contiguous tensor on the device or, where pinned memory is
// allowed, pinned; false: not such a tensor.
bool any_count(PyObject* o, Kind kind, void** p, bool pinned_ok = false) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!dtype_is(t.scalar_type(), kind) || !t.is_contiguous()) return false;
  if (!t.is_cuda() && !(pinned_ok && t.is_pinned())) return false;
  *p = t.data_ptr();
  return true;
}
// The same, of exactly n elements.
bool tensor(PyObject* o, int64_t n, Kind kind, void** p, bool pinned_ok = false) {
  return THPVariable_CheckExact(o) && THPVariable_Unpack(o).numel() == n && any_count(o, kind, p, pinned_ok);
}

bool int32(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}

// The dims structure (its address, taken by the binding) and the stream: a handle or None, the current stream.
const oasis_dims* dims_at(PyObject* o) { return static_cast<const oasis_dims*>(PyLong_AsVoidPtr(o)); }
bool stream_at(PyObject* o, void** s) {
  if (o == Py_None) {
    *s = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  if (!PyLong_CheckExact(o)) return false;
  *s = PyLong_AsVoidPtr(o);
  return !PyErr_Occurred();
}

#define FALLBACK             \
  do {                       \
    if (PyErr_Occurred()) PyErr_Clear(); \
    Py_RETURN_NONE;          \
  } while (0)

// Runs `call` without the GIL (a full queue blocks the launch) and returns its status.
template <typename F>
PyObject* run(F&& call) {
  oasis_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)st);
}

// No C++ exception (a tensor without storage throws) leaves an entry.
template <typename F>
PyObject* guarded(F&& body) {
  try {
    return body();
  } catch (...) {
    FALLBACK;
  }
}

using Args = PyObject* const*;

// dims, q, num_q_tokens, pool_k, pool_v, slot_map, k_slots, ctx_len, scale, out, lse, workspace, stream
PyObject* sparse_decode_attn(PyObject*, Args a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 13) FALLBACK;
    const oasis_dims* d = dims_at(a[0]);
    int32_t T, k;
    if (!d || !int32(a[2], &T) || !int32(a[6], &k)) FALLBACK;
    const int64_t R = d->num_reqs, H = d->num_kv_heads, D = d->head_dim;
    const int64_t rows = count({R, T, d->num_q_heads}), qn = count({R, T, d->num_q_heads, D});
    const int64_t pool = count({R, (int64_t)k + 1, H, d->block_size, D});
    void *q, *pk, *pv, *map, *ctx, *out, *lse = nullptr, *ws, *s;
    float scale;
    if (D <= 0) FALLBACK;  // no default scale
    if (a[8] == Py_None) scale = (float)(1.0 / std::sqrt((double)D));
    else if (PyFloat_CheckExact(a[8])) scale = (float)PyFloat_AS_DOUBLE(a[8]);
    else FALLBACK;
    if (!tensor(a[1], qn, kBf16, &q) || !tensor(a[3], pool, kBf16, &pk) || !tensor(a[4], pool, kBf16, &pv) ||
        !tensor(a[5], count({R, H, k}), kI32, &map) || !tensor(a[7], R, kI32, &ctx) || !tensor(a[9], qn, kBf16, &out) ||
        (a[10] != Py_None && !tensor(a[10], rows, kF32, &lse)) || !any_count(a[11], kU8, &ws) ||
        !stream_at(a[12], &s))
      FALLBACK;
    const size_t bytes = (size_t)THPVariable_Unpack(a[11]).numel();
    return run([&] {
      return f_attn(d, (const uint16_t*)q, T, (const uint16_t*)pk, (const uint16_t*)pv, (const int32_t*)map, k,
                    (const int32_t*)ctx, scale, (uint16_t*)out, (float*)lse, ws, bytes, s);
    });
  });
}

struct Score {
  int32_t T, first, num;
  void *q, *kmax, *kmin, *ctx, *scores;
};
// q, num_q_tokens, first_draft, num_draft, kmax, kmin, ctx_len at a[1..7]; scores at a[scores]
bool score_args(const oasis_dims* d, Args a, int scores, Score* s) {
  if (!d || !int32(a[2], &s->T) || !int32(a[3], &s->first) || !int32(a[4], &s->num)) return false;
  const int64_t R = d->num_reqs, H = d->num_kv_heads, NB = d->max_blocks, D = d->head_dim;
  const int64_t summary = count({R, H, NB, D});
  return tensor(a[1], count({R, s->T, d->num_q_heads, D}), kBf16, &s->q) && tensor(a[5], summary, kBf16, &s->kmax) &&
         tensor(a[6], summary, kBf16, &s->kmin) && tensor(a[7], R, kI32, &s->ctx) &&
         tensor(a[scores], count({R, H, NB}), kF32, &s->scores);
}

// dims, q, num_q_tokens, first_draft, num_draft, kmax, kmin, ctx_len, scores, stream
PyObject* score_blocks(PyObject*, Args a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 10) FALLBACK;
    const oasis_dims* d = dims_at(a[0]);
    Score c;
    void* s;
    if (!score_args(d, a, 8, &c) || !stream_at(a[9], &s)) FALLBACK;
    return run([&] {
      return f_score(d, (const uint16_t*)c.q, c.T, c.first, c.num, (const uint16_t*)c.kmax, (const uint16_t*)c.kmin,
                     (const int32_t*)c.ctx, (float*)c.scores, s);
    });
  });
}

// dims, scores, ctx_len, k, sel, sel_count, stream
PyObject* select_topk(PyObject*, Args a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 7) FALLBACK;
    const oasis_dims* d = dims_at(a[0]);
    int32_t k;
    void *scores, *ctx, *sel, *cnt, *s;
    if (!d || !int32(a[3], &k)) FALLBACK;
    const int64_t R = d->num_reqs, RH = count({R, d->num_kv_heads});
    if (!tensor(a[1], count({RH, d->max_blocks}), kF32, &scores) || !tensor(a[2], R, kI32, &ctx) ||
        !tensor(a[4], count({RH, k}), kI32, &sel) || !tensor(a[5], RH, kI32, &cnt) || !stream_at(a[6], &s))
      FALLBACK;
    return run([&] {
      return f_topk(d, (const float*)scores, (const int32_t*)ctx, k, (int32_t*)sel, (int32_t*)cnt, s);
    });
  });
}

// dims, q, num_q_tokens, first_draft, num_draft, kmax, kmin, ctx_len, k, scores, sel, sel_count, stream
PyObject* score_select(PyObject*, Args a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 13) FALLBACK;
    const oasis_dims* d = dims_at(a[0]);
    Score c;
    int32_t k;
    void *sel, *cnt, *s;
    if (!score_args(d, a, 9, &c) || !int32(a[8], &k)) FALLBACK;
    const int64_t RH = count({d->num_reqs, d->num_kv_heads});
    if (!tensor(a[10], count({RH, k}), kI32, &sel) || !tensor(a[11], RH, kI32, &cnt) || !stream_at(a[12], &s)) FALLBACK;
    return run([&] {
      return f_score_select(d, (const uint16_t*)c.q, c.T, c.first, c.num, (const uint16_t*)c.kmax,
                            (const uint16_t*)c.kmin, (const int32_t*)c.ctx, k, (float*)c.scores, (int32_t*)sel,
                            (int32_t*)cnt, s);
    });
  });
}

// dims, host_k, host_v, num_pages, host_block_table, ctx_len, sel, sel_count, scores, k, slot_map, slot_stamp, step,
// fetch_cap, copy_local, pool_k, pool_v, moved, stream
PyObject* stage_blocks(PyObject*, Args a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 19) FALLBACK;
    const oasis_dims* d = dims_at(a[0]);
    int32_t pages, k, step, cap;
    if (!d || !int32(a[3], &pages) || !int32(a[9], &k) || !int32(a[12], &step) || !int32(a[13], &cap) ||
        (a[14] != Py_True && a[14] != Py_False))
      FALLBACK;
    const int64_t R = d->num_reqs, H = d->num_kv_heads, RH = count({R, H});
    const int64_t tier = count({pages, H, d->block_size, d->head_dim});
    const int64_t pool = count({RH, (int64_t)k + 1, d->block_size, d->head_dim}), items = count({RH, k});
    void *hk, *hv, *table, *ctx, *sel, *cnt, *scores, *map, *stamp, *pk, *pv, *moved, *s;
    if (!tensor(a[1], tier, kBf16, &hk, true) || !tensor(a[2], tier, kBf16, &hv, true) ||
        !tensor(a[4], count({R, d->max_blocks}), kI32, &table) || !tensor(a[5], R, kI32, &ctx) ||
        !tensor(a[6], items, kI32, &sel) || !tensor(a[7], RH, kI32, &cnt) ||
        !tensor(a[8], count({RH, d->max_blocks}), kF32, &scores) || !tensor(a[10], items, kI32, &map) ||
        !tensor(a[11], items, kI32, &stamp) || !tensor(a[15], pool, kBf16, &pk) ||
        !tensor(a[16], pool, kBf16, &pv) || !tensor(a[17], RH, kI32, &moved) || !stream_at(a[18], &s))
      FALLBACK;
    const int32_t copy_local = a[14] == Py_True;
    return run([&] {
      return f_stage(d, (const uint16_t*)hk, (const uint16_t*)hv, pages, (const int32_t*)table, (const int32_t*)ctx,
                     (const int32_t*)sel, (const int32_t*)cnt, (const float*)scores, k, (int32_t*)map,
                     (int32_t*)stamp, step, cap, copy_local, (uint16_t*)pk, (uint16_t*)pv, (int32_t*)moved, s);
    });
  });
}

// bind(attn, score, topk, score_select, stage): addresses of the library's entry points
PyObject* bind(PyObject*, Args a, Py_ssize_t n) {
  void* p[5];
  if (n != 5) return PyErr_Format(PyExc_TypeError, "bind takes 5 addresses");
  for (int i = 0; i < 5; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "bind: null address");
  }
  f_attn = reinterpret_cast<decltype(f_attn)>(p[0]);
  f_score = reinterpret_cast<decltype(f_score)>(p[1]);
  f_topk = reinterpret_cast<decltype(f_topk)>(p[2]);
  f_score_select = reinterpret_cast<decltype(f_score_select)>(p[3]);
  f_stage = reinterpret_cast<decltype(f_stage)>(p[4]);
  Py_RETURN_NONE;
}

#define METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind),         METHOD(sparse_decode_attn), METHOD(score_blocks), METHOD(select_topk),
                         METHOD(score_select), METHOD(stage_blocks),       {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
  PyObject* m = PyModule_Create(&module);
  // the signatures the calls above were compiled with; the binding compares it with the loaded library's
  if (m && PyModule_AddIntConstant(m, "abi_version", OASIS_ABI_VERSION) < 0) Py_CLEAR(m);
  return m;
}
