// The per-chunk calls from Python without ctypes.  One pass of a small chunk is two calls, and marshalling their
// two dozen arguments through ctypes took 9 to 11 us of each where the launch itself takes 2 to 3.
//
// Every function here takes the arguments of its namesake in binding.py in C order, the stream as an integer, and
// returns the C function's result.  It handles plain arguments only (torch.Tensor, int, float, a list of
// pairs) and returns NotImplemented for anything else, a tensor of another rank or stride, and whatever makes the
// tensor's own accessors throw: binding.py then takes its general path, which raises what it always raised.
// Nothing is kept between calls but the addresses of the library's functions and the descriptor's type.
#include <Python.h>
#include <ATen/core/TensorBase.h>
#include <torch/csrc/autograd/python_variable.h>
#include "../../include/crope.h"

// The torch and Python that this is compiled for (build.py): looked for in the file before it is loaded.
extern "C" __attribute__((visibility("default"), used)) const char crope_fastcall_for[] = CROPE_FASTCALL_FOR;

namespace {

decltype(&crope_qk_norm_rotate_append) p_append;
decltype(&crope_qk_norm_rotate_append_qscaled) p_append_qscaled;
decltype(&chunk_attention) p_attention;
decltype(&chunk_attention_planned) p_attention_planned;
decltype(&chunk_attention_static) p_attention_static;
decltype(&chunk_attention_limited) p_attention_limited;
decltype(&crope_qkv_project_norm_rotate_append) p_project;
PyObject* g_desc_type;
PyObject* g_field[8];
constexpr int kMaxSegs = 16;   // more than the library takes

// One call's arguments, read from left to right; `ok` turns false at the first that is not plain.
struct Reader {
  PyObject* const* args;
  Py_ssize_t n, i = 0;
  bool ok = true;

  PyObject* next() {
    if (i >= n) { ok = false; return nullptr; }
    return args[i++];
  }
  int64_t integer(int64_t lo, int64_t hi) {
    PyObject* o = next();
    if (!ok || !PyLong_CheckExact(o)) { ok = false; return 0; }
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    if (over || v < lo || v > hi) { ok = false; return 0; }
    return v;
  }
  int32_t i32() { return (int32_t)integer(INT32_MIN, INT32_MAX); }
  int64_t i64() { return integer(INT64_MIN, INT64_MAX); }
  size_t size() { return (size_t)integer(0, INT64_MAX); }
  void* stream() {
    if (ok && i < n && args[i] == Py_None) { ++i; return nullptr; }
    return (void*)(uintptr_t)integer(0, INT64_MAX);
  }
  float f32() {
    PyObject* o = next();
    if (!ok || !PyFloat_CheckExact(o)) { ok = false; return 0.f; }
    return (float)PyFloat_AS_DOUBLE(o);
  }
  const at::Tensor* tensor() {
    PyObject* o = next();
    if (!ok || !THPVariable_CheckExact(o)) { ok = false; return nullptr; }
    return &THPVariable_Unpack(o);
  }
  void* ptr() {
    const at::Tensor* t = tensor();
    return ok ? t->data_ptr() : nullptr;
  }
  void* ptr_or_null() {
    if (ok && i < n && args[i] == Py_None) { ++i; return nullptr; }
    return ptr();
  }
  // a [token][head][128] tensor with contiguous channels
  void* rows(crope_strides* s) {
    const at::Tensor* t = tensor();
    if (!ok || t->dim() != 3 || t->stride(2) != 1) { ok = false; return nullptr; }
    s->token = t->stride(0);
    s->head = t->stride(1);
    return t->data_ptr();
  }
  void* rows_like(const crope_strides& s) {
    crope_strides own;
    void* p = rows(&own);
    if (ok && (own.token != s.token || own.head != s.head)) ok = false;
    return p;
  }
  crope_table_desc desc() {
    crope_table_desc d{};
    PyObject* o = next();
    if (!ok || (PyObject*)Py_TYPE(o) != g_desc_type) { ok = false; return d; }
    int32_t* const ints[7] = {&d.head_dim, &d.dim_t, &d.dim_h, &d.dim_w, &d.max_t, &d.max_h, &d.max_w};
    for (int k = 0; k < 8 && ok; ++k) {
      PyObject* v = PyObject_GetAttr(o, g_field[k]);
      if (!v) { PyErr_Clear(); ok = false; break; }
      if (k == 7) {
        if (PyFloat_CheckExact(v)) d.theta = PyFloat_AS_DOUBLE(v); else ok = false;
      } else {
        Reader one{&v, 1};
        *ints[k] = one.i32();
        ok = one.ok;
      }
      Py_DECREF(v);
    }
    return d;
  }
  int32_t segments(crope_kv_segment* out) {
    PyObject* o = next();
    if (!ok || !PyList_CheckExact(o) || PyList_GET_SIZE(o) > kMaxSegs) { ok = false; return 0; }
    const Py_ssize_t m = PyList_GET_SIZE(o);
    for (Py_ssize_t k = 0; k < m && ok; ++k) {
      PyObject* pair = PyList_GET_ITEM(o, k);
      if (!PyTuple_CheckExact(pair) || PyTuple_GET_SIZE(pair) != 2) { ok = false; break; }
      Reader r{reinterpret_cast<PyTupleObject*>(pair)->ob_item, 2};
      out[k].start = r.i64();
      out[k].len = r.i64();
      ok = r.ok;
    }
    return (int32_t)m;
  }
  bool done() const { return ok && i == n; }
};

PyObject* not_plain() { Py_RETURN_NOTIMPLEMENTED; }

template <class F>
PyObject* call(F f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

template <bool SCALED>
PyObject* append_impl(PyObject* const* args, Py_ssize_t n) {
  Reader r{args, n};
  const crope_table_desc d = r.desc();
  const float* table = (const float*)r.ptr();
  crope_strides in, qo, c;
  void *q = r.rows(&in), *k = r.rows_like(in), *v = r.rows_like(in);
  const float *gq = (const float*)r.ptr(), *gk = (const float*)r.ptr();
  const float eps = r.f32();
  const int32_t group = r.i32(), tokens = r.i32(), heads = r.i32(), gh = r.i32(), gw = r.i32(), start = r.i32(), off = r.i32();
  const float q_scale = SCALED ? r.f32() : 1.0f;
  void *q_out = r.rows(&qo), *kc = r.rows(&c), *vc = r.rows_like(c);
  const int64_t cap = r.i64(), dst = r.i64();
  void* st = r.stream();
  if (!r.done()) return not_plain();
  if (SCALED)
    return call([&] { return p_append_qscaled(&d, table, q, k, v, in, gq, gk, eps, group, tokens, heads, gh, gw, start, off,
                                              q_scale, q_out, qo, kc, vc, c, cap, dst, st); });
  return call([&] { return p_append(&d, table, q, k, v, in, gq, gk, eps, group, tokens, heads, gh, gw, start, off, q_out, qo, kc,
                                    vc, c, cap, dst, st); });
}

enum Kind { kOwnWorkspace, kPlanned, kStatic, kLimited };

template <Kind K>
PyObject* attention_impl(PyObject* const* args, Py_ssize_t n) {
  Reader r{args, n};
  crope_strides qs, c, os;
  crope_kv_segment segs[kMaxSegs];
  void* q = r.rows(&qs);
  const int32_t n_q = r.i32(), heads = r.i32();
  void *kc = r.rows(&c), *vc = r.rows_like(c);
  const int64_t cap = r.i64();
  const int32_t n_segs = r.segments(segs);
  const float scale = r.f32();
  crope_attention_plan plan{0, 0};
  if (K == kPlanned) {
    plan.waves = r.i32();
    plan.splits = r.i32();
  }
  const int32_t* limit = K == kLimited ? (const int32_t*)r.ptr() : nullptr;
  void* out = r.rows(&os);
  float* lse = (float*)r.ptr_or_null();
  void* ws = K == kOwnWorkspace || K == kPlanned ? r.ptr_or_null() : nullptr;
  const size_t ws_bytes = K == kOwnWorkspace || K == kPlanned ? r.size() : 0;
  void* st = r.stream();
  if (!r.done()) return not_plain();
  return call([&] {
    switch (K) {
      case kOwnWorkspace: return p_attention(q, qs, n_q, heads, kc, vc, c, cap, segs, n_segs, scale, out, os, lse, ws, ws_bytes, st);
      case kPlanned: return p_attention_planned(q, qs, n_q, heads, kc, vc, c, cap, segs, n_segs, scale, &plan, out, os, lse, ws, ws_bytes, st);
      case kStatic: return p_attention_static(q, qs, n_q, heads, kc, vc, c, cap, segs, n_segs, scale, out, os, lse, st);
      default: return p_attention_limited(q, qs, n_q, heads, kc, vc, c, cap, segs, n_segs, scale, limit, out, os, lse, st);
    }
  });
}

PyObject* project_impl(PyObject* const* args, Py_ssize_t n) {
  Reader r{args, n};
  const crope_table_desc d = r.desc();
  const float* table = (const float*)r.ptr();
  const at::Tensor* x = r.tensor();
  if (r.ok && (x->dim() != 2 || x->stride(1) != 1)) r.ok = false;
  const at::Tensor* w = r.tensor();
  if (r.ok && (w->dim() != 2 || !w->is_contiguous())) r.ok = false;
  const float* bias = (const float*)r.ptr_or_null();
  const int32_t c_in = r.i32();
  const float *gq = (const float*)r.ptr(), *gk = (const float*)r.ptr();
  const float eps = r.f32();
  const int32_t group = r.i32(), tokens = r.i32(), heads = r.i32(), gh = r.i32(), gw = r.i32(), start = r.i32(), off = r.i32();
  crope_strides qo, c;
  void *q_out = r.rows(&qo), *kc = r.rows(&c), *vc = r.rows_like(c);
  const int64_t cap = r.i64(), dst = r.i64();
  void* ws = r.ptr_or_null();
  const size_t ws_bytes = r.size();
  void* st = r.stream();
  if (!r.done()) return not_plain();
  const void *xp = x->data_ptr(), *wp = w->data_ptr();
  const int64_t x_stride = x->stride(0);
  return call([&] { return p_project(&d, table, xp, x_stride, wp, bias, c_in, gq, gk, eps, group, tokens, heads, gh, gw, start, off,
                                     q_out, qo, kc, vc, c, cap, dst, ws, ws_bytes, st); });
}

// a tensor without ordinary storage (a wrapper of a functional transform, say) throws in its accessors
template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* args, Py_ssize_t n) {
  try {
    return F(args, n);
  } catch (...) {
    PyErr_Clear();
    return not_plain();
  }
}

// bind(addresses, TableDesc): the library's functions, in the order of the pointers above
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *list, *type;
  if (!PyArg_ParseTuple(args, "O!O", &PyList_Type, &list, &type)) return nullptr;
  if (PyList_GET_SIZE(list) != 7) { PyErr_SetString(PyExc_ValueError, "seven addresses expected"); return nullptr; }
  void* a[7];
  for (int k = 0; k < 7; ++k) {
    a[k] = PyLong_AsVoidPtr(PyList_GET_ITEM(list, k));
    if (!a[k]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  p_append = (decltype(p_append))a[0];
  p_append_qscaled = (decltype(p_append_qscaled))a[1];
  p_attention = (decltype(p_attention))a[2];
  p_attention_planned = (decltype(p_attention_planned))a[3];
  p_attention_static = (decltype(p_attention_static))a[4];
  p_attention_limited = (decltype(p_attention_limited))a[5];
  p_project = (decltype(p_project))a[6];
  Py_INCREF(type);
  Py_XSETREF(g_desc_type, type);
  Py_RETURN_NONE;
}

#define FAST(name, f) {name, (PyCFunction)(void*)&guarded<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    FAST("append", append_impl<false>),
    FAST("append_qscaled", append_impl<true>),
    FAST("attention", attention_impl<kOwnWorkspace>),
    FAST("attention_planned", attention_impl<kPlanned>),
    FAST("attention_static", attention_impl<kStatic>),
    FAST("attention_limited", attention_impl<kLimited>),
    FAST("project", project_impl),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
  const char* names[8] = {"head_dim", "dim_t", "dim_h", "dim_w", "max_t", "max_h", "max_w", "theta"};
  for (int k = 0; k < 8; ++k)
    if (!(g_field[k] = PyUnicode_InternFromString(names[k]))) return nullptr;
  return PyModule_Create(&module);
}
