// The calls of a training step from Python: tensors, list headers and the current stream -> the C ABI of include/lx.h.
//
// The smallest calls take the GPU two to five microseconds, and the host as much: a launch alone 2.8 - 3.6 us, and what is done
// for a call in Python, through ctypes / here, us, with C functions that return at once: a mask's list 1.85 / 0.77, FFN forward and
// backward 2.1 and 2.2 / 1.0 and 1.1, attention, whose tensors' strides are compared, 3.05 and 4.4 / 1.6 and 2.55, LoRA backward 3.0 /
// 1.5, predictor 1.7 / 0.95.
// Host time, us, through ctypes and so: one list and two FFN calls of two launches each 22.9 -> 19.6, lists and both attention
// calls 21.6 -> 16.3, a LoRA pass of nine launches 34.1 -> 29.8.  Whole passes of 24 and 21 us become 1.06 and 1.09 times as fast (with
// the compaction's share), long ones wait for the GPU.
//
// Every argument is read when the call is made, through the same attributes and methods of the tensor that Python code would
// use (data_ptr, shape, stride, dtype, numel); nothing about a tensor is kept.  The library's functions are handed over by
// address (bind), so this module belongs to the library that loaded it.  Numbers are converted as the C prototypes in ctypes
// convert them: integers modulo 2^32, ctypes' own objects and what `_as_parameter_` holds through `types`' converter, and
// everything else is its ArgumentError; last of all, after what is refused for other reasons.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include <type_traits>

#include "../../include/lx.h"

namespace {

// Of one module object: every copy of the binding has its own.  Set by bind and types.
struct State {
  decltype(&lx_mask_compact) mask_compact;
  decltype(&lx_mask_compact_pair) mask_compact_pair;
  decltype(&lx_attn_combine_patterns) combine;
  decltype(&lx_mlp_predict_mask) predict;
  decltype(&lx_sparse_ffn_fwd) ffn_fwd;
  decltype(&lx_sparse_ffn_bwd_dx) ffn_bwd;
  decltype(&lx_sparse_ffn_lora_fwd) lora_fwd;
  decltype(&lx_sparse_ffn_lora_bwd) lora_bwd;
  decltype(&lx_sparse_attn_fwd) attn_fwd;
  decltype(&lx_sparse_attn_bwd_dx) attn_bwd;
  decltype(&lx_sparse_attn_bwd_dx_noalloc) attn_bwd_noalloc;
  PyObject *dtypes, *error, *stream, *uint8, *float32, *int32;     // {torch dtype: lx_dtype}, LxError, () -> raw stream, torch dtypes
  PyObject *list, *i32, *f32, *convert, *wrong;    // list header, c_int32, c_float, (value, type) -> number, the error of wrong types
};
constexpr PyObject* State::*kHeld[] = {&State::dtypes, &State::error, &State::stream, &State::uint8, &State::float32, &State::int32,
                                       &State::list, &State::i32, &State::f32, &State::convert, &State::wrong};
State& state(PyObject* module) { return *static_cast<State*>(PyModule_GetState(module)); }
struct Names {
  PyObject *data_ptr, *shape, *stride, *dtype, *numel, *element_size, *is_cuda, *is_contiguous;
} n;

// An error is pending once `bad` is set; what follows is then skipped by the callers' single test before the call.
struct Args {
  const State& g;
  PyObject* const* a;
  bool bad = false;
  Py_buffer header[4];
  int headers = 0;
  Args(const State& state, PyObject* const* args) : g(state), a(args) {}
  ~Args() {
    for (int i = 0; i < headers; ++i) PyBuffer_Release(&header[i]);
  }
  void require(bool ok) {
    if (!bad && !ok) {
      bad = true;
      if (!PyErr_Occurred()) PyErr_SetNone(PyExc_AssertionError);
    }
  }
  void wrong(const char* what, PyObject* o) {
    bad = true;
    PyErr_Format(g.wrong, "%s expected, got %s", what, Py_TYPE(o)->tp_name);
  }
  // Of an integer; of anything else what `convert` makes of it.
  long long number(PyObject* o) {
    if (bad) return 0;
    if (PyLong_Check(o)) return (long long)PyLong_AsUnsignedLongLongMask(o);
    PyObject* r = PyObject_CallFunctionObjArgs(g.convert, o, g.i32, nullptr);
    const long long v = r ? PyLong_AsLongLong(r) : -1;
    Py_XDECREF(r);
    bad |= v == -1 && PyErr_Occurred();
    return v;
  }
  int32_t number(int i) { return (int32_t)number(a[i]); }
  float real(int i) {
    if (bad) return 0;
    if (PyFloat_Check(a[i])) return (float)PyFloat_AS_DOUBLE(a[i]);
    PyObject* r = PyObject_CallFunctionObjArgs(g.convert, a[i], g.f32, nullptr);
    const double v = r ? PyFloat_AsDouble(r) : -1.0;
    Py_XDECREF(r);
    bad |= v == -1.0 && PyErr_Occurred();
    return (float)v;
  }
  void* address(PyObject* r) {          // of a number or None; releases it
    if (!r) return bad = true, nullptr;
    void* p = nullptr;
    if (PyLong_Check(r))
      p = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(r));
    else if (r != Py_None)
      wrong("address", r);
    Py_DECREF(r);
    return p;
  }
  bool truth(int i) {
    const int v = bad ? 0 : PyObject_IsTrue(a[i]);
    bad |= v < 0;
    return v > 0;
  }
  // Results of a method or an attribute as numbers.
  long long method(int i, PyObject* name) {
    PyObject* r = bad ? nullptr : PyObject_CallMethodNoArgs(a[i], name);
    if (!r) return bad = true, 0;
    const long long v = number(r);
    Py_DECREF(r);
    return v;
  }
  bool flag(PyObject* r) {
    if (!r) return bad = true, false;
    const int v = PyObject_IsTrue(r);
    Py_DECREF(r);
    bad |= v < 0;
    return v > 0;
  }
  bool is_cuda(int i) { return !bad && flag(PyObject_GetAttr(a[i], n.is_cuda)); }
  bool is_contiguous(int i) { return !bad && flag(PyObject_CallMethodNoArgs(a[i], n.is_contiguous)); }
  void* ptr(int i) {          // of a tensor, or null for None
    if (bad || a[i] == Py_None) return nullptr;
    return address(PyObject_CallMethodNoArgs(a[i], n.data_ptr));
  }
  size_t bytes(int i) { return bad || a[i] == Py_None ? 0 : (size_t)(method(i, n.numel) * method(i, n.element_size)); }
  const lx_blocklist* list(int i) {       // of a ctypes structure, or null for None
    if (bad || a[i] == Py_None) return nullptr;
    const int is = PyObject_IsInstance(a[i], g.list);
    if (is <= 0) {
      bad = true;
      if (is == 0) wrong("list header", a[i]);
      return nullptr;
    }
    if (PyObject_GetBuffer(a[i], &header[headers], PyBUF_SIMPLE) != 0) return bad = true, nullptr;
    return static_cast<const lx_blocklist*>(header[headers++].buf);
  }
  // The numbers of a tuple, at most `most` of them; how many it has, or -1.
  int tuple(PyObject* t, long long* out, int most) {
    if (!t) return bad = true, -1;
    const int len = PyTuple_Check(t) ? (int)PyTuple_GET_SIZE(t) : -1;
    if (len < 0) PyErr_SetString(PyExc_TypeError, "tuple expected"), bad = true;
    for (int k = 0; k < len && k < most && !bad; ++k) out[k] = number(PyTuple_GET_ITEM(t, k));
    Py_DECREF(t);
    return len;
  }
  int shape(int i, long long* out, int most) { return bad ? -1 : tuple(PyObject_GetAttr(a[i], n.shape), out, most); }
  // `want` numbers, with Python's error for unpacking another number of them.
  void unpack(int i, long long* out, int want) {
    const int len = shape(i, out, want);
    if (!bad && len != want) {
      bad = true;
      if (len < want)
        PyErr_Format(PyExc_ValueError, "not enough values to unpack (expected %d, got %d)", want, len);
      else
        PyErr_Format(PyExc_ValueError, "too many values to unpack (expected %d)", want);
    }
  }
  void require_shape(int i, long long x, long long y) {
    long long s[2];
    const int len = shape(i, s, 2);
    if (!bad) require(len == 2 && s[0] == x && s[1] == y);
  }
  long long first(int i) {    // shape[0]
    long long s = 0;
    const int len = shape(i, &s, 1);
    if (!bad && len < 1) PyErr_SetString(PyExc_IndexError, "tuple index out of range"), bad = true;
    return s;
  }
  // The last two sizes of a shape of two and more dimensions, and the product of all.
  long long sizes(int i, long long& x, long long& y) {
    PyObject* t = bad ? nullptr : PyObject_GetAttr(a[i], n.shape);
    if (!t) return bad = true, 0;
    const Py_ssize_t len = PyTuple_Check(t) ? PyTuple_GET_SIZE(t) : 0;
    require(len >= 2);
    long long all = 1;
    for (Py_ssize_t k = 0; k < len && !bad; ++k) x = y, y = number(PyTuple_GET_ITEM(t, k)), all *= y;
    Py_DECREF(t);
    return all;
  }
  void require_dtype(int i, PyObject* want) {
    if (bad) return;
    PyObject* d = PyObject_GetAttr(a[i], n.dtype);
    if (!d) { bad = true; return; }
    const bool same = d == want;        // (torch's dtypes are single objects)
    Py_DECREF(d);
    require(same);
  }
  lx_dtype dtype(int i) {
    if (bad) return LX_F32;
    PyObject* d = PyObject_GetAttr(a[i], n.dtype);
    if (!d) return bad = true, LX_F32;
    PyObject* v = PyDict_GetItemWithError(g.dtypes, d);
    if (!v) {
      bad = true;
      if (!PyErr_Occurred()) {
        PyObject* text = PyUnicode_FromFormat("dtype %S", d);
        if (text) raise(LX_ERR_UNSUPPORTED, text);
        Py_XDECREF(text);
      }
    }
    Py_DECREF(d);
    return v ? (lx_dtype)PyLong_AsLong(v) : LX_F32;
  }
  void* stream() {
    return bad ? nullptr : address(PyObject_CallNoArgs(g.stream));
  }
  void raise(int status, PyObject* where) const {
    PyObject* e = PyObject_CallFunction(g.error, "iO", status, where);
    if (e) PyErr_SetObject(g.error, e);
    Py_XDECREF(e);
  }
};
// Runs `call` without the interpreter lock, as ctypes does.
template <class Call>
PyObject* finish(const Args& a, const char* where, Call call) {
  if (a.bad) return nullptr;
  lx_status s;
  Py_BEGIN_ALLOW_THREADS
  s = call();
  Py_END_ALLOW_THREADS
  if (s == LX_OK) Py_RETURN_NONE;
  if (PyObject* w = PyUnicode_FromString(where)) {
    a.raise(s, w);
    Py_DECREF(w);
  }
  return nullptr;
}
bool count(Py_ssize_t got, Py_ssize_t want) {
  if (got == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, got);
  return false;
}

// A mask tensor [..., R, C], uint8, contiguous, on the GPU: {masks, R, C}.
void mask_shape(Args& a, int i, long long (&m)[3]) {
  a.require_dtype(i, a.g.uint8);
  a.require(a.is_cuda(i));
  a.require(a.is_contiguous(i));
  const long long all = a.sizes(i, m[1], m[2]);
  if (a.bad) return;
  if (m[1] * m[2] == 0) {
    PyErr_SetString(PyExc_ZeroDivisionError, "integer division or modulo by zero");
    a.bad = true;
    return;
  }
  m[0] = all / (m[1] * m[2]);
}

// mask, transpose, nnz_cap or None, row_ptr, col_idx
PyObject* mask_compact(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 5)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long m[3] = {};
  mask_shape(a, 0, m);
  const bool turned = a.truth(1);
  const long long R = m[1], C = m[2];
  const uint8_t* mask = (const uint8_t*)a.ptr(0);
  int32_t *rp = (int32_t*)a.ptr(3), *ci = (int32_t*)a.ptr(4);
  void* st = a.stream();
  const int32_t cap = args[2] != Py_None ? a.number(2) : m[0] > 0 ? (int32_t)(m[0] * R * C) : 1;
  return finish(a, "lx_mask_compact", [&] {
    return g.mask_compact(mask, (int32_t)m[0], (int32_t)(turned ? C : R), (int32_t)(turned ? R : C), R * C, turned ? 1 : C,
                          turned ? C : 1, rp, ci, cap, st);
  });
}
// mask, row_ptr and col_idx of the row list, those of the column list
PyObject* mask_compact_pair(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 5)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long m[3] = {};
  mask_shape(a, 0, m);
  const long long R = m[1], C = m[2];
  const uint8_t* mask = (const uint8_t*)a.ptr(0);
  int32_t* p[4];
  for (int k = 0; k < 4; ++k) p[k] = (int32_t*)a.ptr(1 + k);
  void* st = a.stream();
  return finish(a, "lx_mask_compact_pair", [&] {
    return g.mask_compact_pair(mask, (int32_t)m[0], (int32_t)R, (int32_t)C, R * C, C, 1, p[0], p[1], p[2], p[3], (int32_t)(m[0] * R * C), st);
  });
}
// headers of the pool's row list and of its column list or None, patterns, nblk, head_pattern, nnz_cap, row_ptr, col_idx of the
// row list, those of the column list or None
PyObject* combine(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 10)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  a.require_dtype(4, g.int32);
  a.require(a.is_cuda(4));
  a.require(a.is_contiguous(4));
  const lx_blocklist *r = a.list(0), *c = a.list(1);
  const int32_t heads = (int32_t)a.method(4, n.numel);
  const int32_t* hp = (const int32_t*)a.ptr(4);
  int32_t* p[4];
  for (int k = 0; k < 4; ++k) p[k] = (int32_t*)a.ptr(6 + k);
  void* st = a.stream();
  const int32_t P = a.number(2), nblk = a.number(3), cap = a.number(5);
  return finish(a, "lx_attn_combine_patterns", [&] { return g.combine(r, c, P, nblk, hp, heads, p[0], p[1], p[2], p[3], cap, st); });
}
// X, Wa_t, thr, group_rows, mask
PyObject* predict(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 5)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long x[2] = {};
  a.unpack(0, x, 2);
  const long long nblk = a.first(1);
  a.require_shape(1, nblk, x[1]);
  a.require(a.is_contiguous(0));
  a.require(a.is_contiguous(1));
  const lx_dtype dt = a.dtype(0);
  const void *X = a.ptr(0), *W = a.ptr(1);
  uint8_t* mask = (uint8_t*)a.ptr(4);
  void* st = a.stream();
  const int32_t group = a.number(3);
  const float thr = a.real(2);
  return finish(a, "lx_mlp_predict_mask", [&] { return g.predict(dt, (int32_t)x[0], (int32_t)x[1], (int32_t)nblk, group, X, W, thr, mask, st); });
}
// X, W_up, W_down, header, tile_t, blk_n, Y, H_act, b_up, b_down, workspace
PyObject* ffn_fwd(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 11)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long x[2] = {};
  a.unpack(0, x, 2);
  const int32_t F = (int32_t)a.first(1);
  const size_t ws_bytes = a.bytes(10);
  const lx_dtype dt = a.dtype(0);
  const void *X = a.ptr(0), *Wu = a.ptr(1), *bu = a.ptr(8), *Wd = a.ptr(2), *bd = a.ptr(9);
  void *Y = a.ptr(6), *H = a.ptr(7), *ws = a.ptr(10), *st = a.stream();
  const int32_t tt = a.number(4), bn = a.number(5);
  const lx_blocklist* bl = a.list(3);
  return finish(a, "lx_sparse_ffn_fwd", [&] {
    return g.ffn_fwd(dt, (int32_t)x[0], (int32_t)x[1], F, tt, bn, X, Wu, bu, Wd, bd, bl, Y, H, ws, ws_bytes, st);
  });
}
// dY, H_act, W_up, W_down, header, tile_t, blk_n, dX, workspace, W_up_t, W_down_t
PyObject* ffn_bwd(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 11)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long x[2] = {};
  a.unpack(0, x, 2);
  const int32_t F = (int32_t)a.first(args[2] != Py_None ? 2 : 10);
  const size_t ws_bytes = a.bytes(8);
  const lx_dtype dt = a.dtype(0);
  const void *dY = a.ptr(0), *H = a.ptr(1), *Wu = a.ptr(2), *Wd = a.ptr(3), *Wut = a.ptr(9), *Wdt = a.ptr(10);
  void *dX = a.ptr(7), *ws = a.ptr(8), *st = a.stream();
  const int32_t tt = a.number(5), bn = a.number(6);
  const lx_blocklist* bl = a.list(4);
  return finish(a, "lx_sparse_ffn_bwd_dx", [&] {
    return g.ffn_bwd(dt, (int32_t)x[0], (int32_t)x[1], F, tt, bn, dY, H, Wu, Wd, Wut, Wdt, bl, dX, ws, ws_bytes, st);
  });
}
// X, W_up, A_pad, B_pad, W_down, header, Y, H_act, U, workspace
PyObject* lora_fwd(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 10)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long x[2] = {};
  a.unpack(0, x, 2);
  const long long F = a.first(1);
  a.require_shape(2, 64, x[1]);
  a.require_shape(3, F, 64);
  a.require_shape(8, x[0], 64);
  const lx_dtype dt = a.dtype(0);
  const size_t ws_bytes = a.bad ? 0 : (size_t)a.method(9, n.numel);
  const void *X = a.ptr(0), *Wu = a.ptr(1), *A = a.ptr(2), *B = a.ptr(3), *Wd = a.ptr(4);
  void *Y = a.ptr(6), *H = a.ptr(7), *U = a.ptr(8), *ws = a.ptr(9), *st = a.stream();
  const lx_blocklist* bl = a.list(5);
  return finish(a, "lx_sparse_ffn_lora_fwd", [&] {
    return g.lora_fwd(dt, (int32_t)x[0], (int32_t)x[1], (int32_t)F, 64, 64, X, Wu, A, B, Wd, bl, Y, H, U, ws, ws_bytes, st);
  });
}
// X, dY, H_act, U, W_up_t, W_down_t, A_pad, B_pad, header, dX, dA, dB, workspace
PyObject* lora_bwd(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 13)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long x[2] = {};
  a.unpack(0, x, 2);
  const long long F = a.first(5);
  a.require_dtype(10, g.float32);
  a.require_shape(10, 64, x[1]);
  a.require_dtype(11, g.float32);
  a.require_shape(11, F, 64);
  a.require_shape(4, x[1], F);
  a.require_shape(5, F, x[1]);
  const lx_dtype dt = a.dtype(0);
  const size_t ws_bytes = a.bad ? 0 : (size_t)a.method(12, n.numel);
  const void *X = a.ptr(0), *dY = a.ptr(1), *H = a.ptr(2), *U = a.ptr(3), *Wut = a.ptr(4), *Wdt = a.ptr(5), *A = a.ptr(6), *B = a.ptr(7);
  float *dA = (float*)a.ptr(10), *dB = (float*)a.ptr(11);
  void *dX = a.ptr(9), *ws = a.ptr(12), *st = a.stream();
  const lx_blocklist* bl = a.list(8);
  return finish(a, "lx_sparse_ffn_lora_bwd", [&] {
    return g.lora_bwd(dt, (int32_t)x[0], (int32_t)x[1], (int32_t)F, 64, 64, X, dY, H, U, Wut, Wdt, A, B, bl, dX, dA, dB, ws, ws_bytes, st);
  });
}

// Shape of Q and the first three element strides, which the tensors at `others` share with it.
void attn_shape(Args& a, const int* others, int count, long long (&q)[4], int64_t (&st)[3]) {
  a.unpack(0, q, 4);
  PyObject* shape = a.bad ? nullptr : PyObject_GetAttr(a.a[0], n.shape);
  PyObject* stride = shape ? PyObject_CallMethodNoArgs(a.a[0], n.stride) : nullptr;
  a.bad |= !stride;
  for (int k = 0; k < count && !a.bad; ++k) {
    PyObject* t = a.a[others[k]];
    PyObject* s = PyObject_CallMethodNoArgs(t, n.stride);
    int same = s ? PyObject_RichCompareBool(s, stride, Py_EQ) : -1;
    Py_XDECREF(s);
    if (same == 1) {
      PyObject* h = PyObject_GetAttr(t, n.shape);
      same = h ? PyObject_RichCompareBool(h, shape, Py_EQ) : -1;
      Py_XDECREF(h);
    }
    if (same < 0) a.bad = true;
    a.require(same == 1);
  }
  if (!a.bad) {
    long long s[4] = {};
    Py_INCREF(stride);
    const int len = a.tuple(stride, s, 4);
    if (!a.bad) a.require(len == 4 && s[3] == 1);
    for (int k = 0; k < 3; ++k) st[k] = s[k];
  }
  Py_XDECREF(shape);
  Py_XDECREF(stride);
}
// Q, K, V, header, scale, causal, O, LSE, mask_batch, head_active
PyObject* attn_fwd(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 10)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  long long q[4] = {};
  int64_t st3[3] = {};
  const int others[] = {1, 2, 6};
  attn_shape(a, others, 3, q, st3);
  const lx_dtype dt = a.dtype(0);
  const void *Q = a.ptr(0), *K = a.ptr(1), *V = a.ptr(2);
  const uint8_t* act = (const uint8_t*)a.ptr(9);
  void* O = a.ptr(6);
  float* LSE = (float*)a.ptr(7);
  void* st = a.stream();
  const float scale = a.real(4);
  const int32_t causal = a.number(5), mb = a.number(8);
  const lx_blocklist* bl = a.list(3);
  return finish(a, "lx_sparse_attn_fwd", [&] {
    return g.attn_fwd(dt, (int32_t)q[0], (int32_t)q[1], (int32_t)q[2], (int32_t)q[3], scale, causal, Q, K, V, st3, bl, mb, act, O, LSE, st);
  });
}
// Q, K, V, O, LSE, dO, header of the row list, of the column list, scale, causal, dQ, dK, dV, workspace, mask_batch, head_active;
// without the workspace: the noalloc call
PyObject* attn_bwd(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  const bool scratch = nargs == 16;
  if (!scratch && !count(nargs, 15)) return nullptr;
  const State& g = state(self);
  Args a(g, args);
  const int after = scratch ? 14 : 13;
  long long q[4] = {};
  int64_t st3[3] = {};
  const int others[] = {1, 2, 3, 5, 10, 11, 12};
  attn_shape(a, others, 7, q, st3);
  const size_t ws_bytes = scratch ? a.bytes(13) : 0;
  const lx_dtype dt = a.dtype(0);
  const void *Q = a.ptr(0), *K = a.ptr(1), *V = a.ptr(2), *O = a.ptr(3), *dO = a.ptr(5);
  const float* LSE = (const float*)a.ptr(4);
  const uint8_t* act = (const uint8_t*)a.ptr(after + 1);
  void *dQ = a.ptr(10), *dK = a.ptr(11), *dV = a.ptr(12), *ws = scratch ? a.ptr(13) : nullptr, *st = a.stream();
  const float scale = a.real(8);
  const int32_t causal = a.number(9), mb = a.number(after);
  const lx_blocklist *rows = a.list(6), *cols = a.list(7);
  const int32_t B = (int32_t)q[0], H = (int32_t)q[1], S = (int32_t)q[2], D = (int32_t)q[3];
  return finish(a, scratch ? "lx_sparse_attn_bwd_dx" : "lx_sparse_attn_bwd_dx_noalloc", [&] {
    return scratch ? g.attn_bwd(dt, B, H, S, D, scale, causal, Q, K, V, O, LSE, dO, st3, rows, cols, mb, act, dQ, dK, dV, ws, ws_bytes, st)
                   : g.attn_bwd_noalloc(dt, B, H, S, D, scale, causal, Q, K, V, O, LSE, dO, st3, rows, cols, mb, act, dQ, dK, dV, st);
  });
}

// The objects of kHeld from `first` on.
void hold(State& g, PyObject* const* from, int first, int n) {
  for (int k = 0; k < n; ++k) {
    PyObject* old = g.*kHeld[first + k];
    Py_INCREF(from[k]);
    g.*kHeld[first + k] = from[k];
    Py_XDECREF(old);
  }
}
// {function name: address}, dtypes, LxError, stream, torch.uint8, torch.float32, torch.int32
PyObject* bind(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 7)) return nullptr;
  State& g = state(self);
  bool ok = true;
  auto take = [&](const char* name, auto& fn) {
    PyObject* v = PyDict_GetItemString(args[0], name);
    void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
    if (!p) {
      if (ok && !PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "%s", name);
      ok = false;
    }
    fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>(p);
  };
  take("lx_mask_compact", g.mask_compact);
  take("lx_mask_compact_pair", g.mask_compact_pair);
  take("lx_attn_combine_patterns", g.combine);
  take("lx_mlp_predict_mask", g.predict);
  take("lx_sparse_ffn_fwd", g.ffn_fwd);
  take("lx_sparse_ffn_bwd_dx", g.ffn_bwd);
  take("lx_sparse_ffn_lora_fwd", g.lora_fwd);
  take("lx_sparse_ffn_lora_bwd", g.lora_bwd);
  take("lx_sparse_attn_fwd", g.attn_fwd);
  take("lx_sparse_attn_bwd_dx", g.attn_bwd);
  take("lx_sparse_attn_bwd_dx_noalloc", g.attn_bwd_noalloc);
  if (!ok) return nullptr;
  hold(g, args + 1, 0, 6);
  Py_RETURN_NONE;
}
// lx_blocklist, c_int32, c_float, converter, error of wrong types
PyObject* types(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  if (!count(nargs, 5)) return nullptr;
  hold(state(self), args, 6, 5);
  Py_RETURN_NONE;
}

#define LX_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {LX_METHOD(bind), LX_METHOD(types), LX_METHOD(mask_compact), LX_METHOD(mask_compact_pair), LX_METHOD(combine), LX_METHOD(predict),
                         LX_METHOD(ffn_fwd), LX_METHOD(ffn_bwd), LX_METHOD(lora_fwd), LX_METHOD(lora_bwd), LX_METHOD(attn_fwd),
                         LX_METHOD(attn_bwd), {nullptr, nullptr, 0, nullptr}};
int visit_held(PyObject* m, visitproc visit, void* arg) {
  for (auto p : kHeld) Py_VISIT(state(m).*p);
  return 0;
}
int clear_held(PyObject* m) {
  for (auto p : kHeld) Py_CLEAR(state(m).*p);
  return 0;
}
int intern_names(PyObject*) {
  struct {
    PyObject** to;
    const char* name;
  } const names[] = {{&n.data_ptr, "data_ptr"}, {&n.shape, "shape"}, {&n.stride, "stride"}, {&n.dtype, "dtype"}, {&n.numel, "numel"},
                     {&n.element_size, "element_size"}, {&n.is_cuda, "is_cuda"}, {&n.is_contiguous, "is_contiguous"}};
  for (const auto& x : names)
    if (!*x.to && !(*x.to = PyUnicode_InternFromString(x.name))) return -1;
  return 0;
}
PyModuleDef_Slot slots[] = {{Py_mod_exec, reinterpret_cast<void*>(intern_names)}, {0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lx_call", nullptr, sizeof(State), methods, slots, visit_held, clear_held, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lx_call() { return PyModuleDef_Init(&module); }
