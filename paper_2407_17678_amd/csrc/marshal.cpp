// The compute calls of binding.py as a CPython extension: tensors become pointers, sizes and strides here instead of in ctypes
// structures.  The smallest calls of this library are shorter than what the interpreter needed to make them (a
// decode step of one short sequence 4.6 us on the GPU, 9.3 through ctypes structures, of which 3.0 to ask torch for its stream object).
//
// A tensor is whatever has torch's methods (data_ptr, stride, shape, is_contiguous, numel, element_size): nothing of torch is
// compiled in, nothing is kept from one call to the next, and what the assertions of the ctypes form refused is refused here in its order.
// The functions return the status of the C entry point; binding.py turns it into an exception.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "../../include/s2attn.h"

namespace {

// Entry points, in the order bind() is given their addresses (_MARSHALLED in binding.py, which compares it with `entry_points`): those of
// the library that ctypes has loaded, so that there is one copy of it in the process.
#define S2_ENTRY_POINTS(X) \
  X(s2_attn_fwd, fwd) X(s2_attn_fwd_rows, fwd_rows) X(s2_attn_fwd_varlen, fwd_varlen) X(s2_attn_bwd_stages, bwd_stages) \
  X(s2_attn_bwd_varlen, bwd_varlen) X(s2_dense_causal_fwd, dense_fwd) X(s2_dense_causal_bwd, dense_bwd) X(s2_attn_decode, decode) \
  X(s2_attn_decode_static, decode_static) X(s2_attn_decode_layout, decode_layout) X(s2_attn_decode_paged, decode_paged) \
  X(s2_attn_decode_paged_layout, decode_paged_layout)
struct Api {
#define X(entry, name) decltype(&entry) name;
  S2_ENTRY_POINTS(X)
#undef X
};
union {
  Api f;
  void* at[sizeof(Api) / sizeof(void*)];
} api;
constexpr Py_ssize_t kEntryPoints = sizeof(Api) / sizeof(void*);

struct Names {
  PyObject *data_ptr, *stride, *shape, *is_contiguous, *numel, *element_size, *value;
} names;

// An owned reference.
struct Ref {
  PyObject* o;
  explicit Ref(PyObject* x) : o(x) {}
  ~Ref() { Py_XDECREF(o); }
  Ref(const Ref&) = delete;
  Ref& operator=(const Ref&) = delete;
};

// All of these return false with an exception set.
bool fail_assert() {
  PyErr_SetNone(PyExc_AssertionError);
  return false;
}
bool as_i64(PyObject* o, int64_t& out) {
  out = PyLong_AsLongLong(o);
  return out != -1 || !PyErr_Occurred();
}
// as a C int argument of ctypes: an integer, its low 32 bits
bool as_i32(PyObject* o, int32_t& out) {
  const Ref i(PyNumber_Index(o));
  if (!i.o) return false;
  out = (int32_t)(uint32_t)PyLong_AsUnsignedLongMask(i.o);
  return !PyErr_Occurred();
}
bool as_float(PyObject* o, float& out) {
  const double x = PyFloat_AsDouble(o);
  out = (float)x;
  return x != -1.0 || !PyErr_Occurred();
}
// a handle or stream: an integer, a ctypes pointer (its `value`) or None
bool as_address(PyObject* o, void*& out) {
  out = nullptr;
  if (o == Py_None) return true;
  if (PyLong_Check(o)) {
    out = PyLong_AsVoidPtr(o);
    return out || !PyErr_Occurred();
  }
  const Ref v(PyObject_GetAttr(o, names.value));
  if (!v.o) return false;
  if (v.o == Py_None) return true;
  out = PyLong_AsVoidPtr(v.o);
  return out || !PyErr_Occurred();
}
template <class T>
bool data_of(PyObject* t, T*& out) {
  out = nullptr;
  if (t == Py_None) return true;
  const Ref p(PyObject_CallMethodNoArgs(t, names.data_ptr));
  if (!p.o) return false;
  out = static_cast<T*>(PyLong_AsVoidPtr(p.o));
  return out || !PyErr_Occurred();
}
bool contiguous(PyObject* t) {
  const Ref c(PyObject_CallMethodNoArgs(t, names.is_contiguous));
  if (!c.o) return false;
  const int yes = PyObject_IsTrue(c.o);
  return yes < 0 ? false : yes ? true : fail_assert();
}
PyObject* strides_of(PyObject* t) {
  PyObject* s = PyObject_CallMethodNoArgs(t, names.stride);
  if (s && !PyTuple_Check(s)) {
    Py_DECREF(s);
    PyErr_SetString(PyExc_TypeError, "stride() gives a tuple");
    return nullptr;
  }
  return s;
}
// the shape, which has to be of `n` sizes (any number: n < 0)
bool sizes_of(PyObject* t, int n, int64_t* out, Py_ssize_t at_least = 0) {
  const Ref s(PyObject_GetAttr(t, names.shape));
  if (!s.o) return false;
  if (!PyTuple_Check(s.o)) {
    PyErr_SetString(PyExc_TypeError, "shape is a tuple");
    return false;
  }
  const Py_ssize_t have = PyTuple_GET_SIZE(s.o);
  if (n >= 0 && have != n) {
    PyErr_Format(PyExc_ValueError, "expected %d sizes, got %zd", n, have);
    return false;
  }
  if (have < at_least) {
    PyErr_SetString(PyExc_IndexError, "tuple index out of range");
    return false;
  }
  for (Py_ssize_t i = 0; i < (n >= 0 ? n : at_least); ++i)
    if (!as_i64(PyTuple_GET_ITEM(s.o, i), out[i])) return false;
  return true;
}
// stride i of a tuple of strides
bool stride_at(PyObject* strides, int i, int64_t& out) {
  if (i >= PyTuple_GET_SIZE(strides)) {
    PyErr_SetString(PyExc_IndexError, "Dimension out of range");
    return false;
  }
  return as_i64(PyTuple_GET_ITEM(strides, i), out);
}
bool unit_stride(PyObject* strides, int i) {
  int64_t s;
  return stride_at(strides, i, s) && (s == 1 || fail_assert());
}
bool same(PyObject* a, PyObject* b) {
  const int eq = PyObject_RichCompareBool(a, b, Py_EQ);
  return eq < 0 ? false : eq ? true : fail_assert();
}

// q, k, v, o, lse and (n == 9) d_o, dq, dk, dv
bool tensors_of(PyObject* const* a, int n, s2_tensors& t) {
  int64_t size[4];
  if (!sizes_of(a[0], 4, size)) return false;
  const Ref qs(strides_of(a[0])), ks(qs.o ? strides_of(a[1]) : nullptr), vs(ks.o ? strides_of(a[2]) : nullptr), os(vs.o ? strides_of(a[3]) : nullptr);
  if (!os.o) return false;
  if (!unit_stride(qs.o, 3) || !unit_stride(ks.o, 3) || !unit_stride(vs.o, 3) || !unit_stride(os.o, 3)) return false;
  if (!same(ks.o, vs.o) || !same(qs.o, os.o)) return false;
  for (int i = 5; i < n; ++i) {
    if (a[i] == Py_None) continue;
    const Ref gs(strides_of(a[i]));
    if (!gs.o || !same(gs.o, i < 7 ? qs.o : ks.o)) return false;
  }
  if (!contiguous(a[4])) return false;
  if (!data_of(a[0], t.q) || !data_of(a[1], t.k) || !data_of(a[2], t.v) || !data_of(a[3], t.o) || !data_of(a[4], t.lse)) return false;
  t.d_o = t.dq = t.dk = t.dv = nullptr;
  if (n == 9 && (!data_of(a[5], t.d_o) || !data_of(a[6], t.dq) || !data_of(a[7], t.dk) || !data_of(a[8], t.dv))) return false;
  t.batch = (int32_t)size[0];
  t.heads = (int32_t)size[1];
  t.seqlen = (int32_t)size[2];
  t.head_dim = (int32_t)size[3];
  return stride_at(qs.o, 0, t.q_stride_b) && stride_at(qs.o, 1, t.q_stride_h) && stride_at(qs.o, 2, t.q_stride_t) &&
         stride_at(ks.o, 0, t.kv_stride_b) && stride_at(ks.o, 1, t.kv_stride_h) && stride_at(ks.o, 2, t.kv_stride_t);
}

bool workspace_of(PyObject* ws, void*& at, size_t& bytes) {
  if (!data_of(ws, at)) return false;
  const Ref n(PyObject_CallMethodNoArgs(ws, names.numel)), e(n.o ? PyObject_CallMethodNoArgs(ws, names.element_size) : nullptr);
  int64_t count, size;
  if (!e.o || !as_i64(n.o, count) || !as_i64(e.o, size)) return false;
  bytes = (size_t)count * (size_t)size;
  return true;
}

// the row offsets of a packed batch: contiguous, n + 1 of them
bool offsets_of(PyObject* cu, PyObject* q, const int32_t*& at, int32_t& num_seqs) {
  int64_t batch;
  if (!sizes_of(q, -1, &batch, 1)) return false;
  if (batch != 1) return fail_assert();
  if (!contiguous(cu)) return false;
  const Ref n(PyObject_CallMethodNoArgs(cu, names.numel));
  int64_t count;
  if (!n.o || !as_i64(n.o, count)) return false;
  if (count < 2) return fail_assert();
  num_seqs = (int32_t)(count - 1);
  return data_of(cu, at);
}

bool count_is(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
  return false;
}

// The call itself, with the interpreter's lock given up (a full queue makes a launch wait).
template <class F>
PyObject* status_of(F&& call) {
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// ------------------------------------------------------------------------------------ calls
// (each: the arguments of the function of the same name in binding.py, the handle or parameters and the stream as addresses)

PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {  // layout, q k v o lse, scale, stream
  s2_tensors t;
  float scale;
  void *layout, *stream;
  if (!count_is(n, 8) || !tensors_of(a + 1, 5, t) || !as_address(a[0], layout) || !as_float(a[6], scale) || !as_address(a[7], stream)) return nullptr;
  return status_of([&] { return api.f.fwd(static_cast<s2_layout*>(layout), &t, scale, stream); });
}

PyObject* fwd_rows(PyObject*, PyObject* const* a, Py_ssize_t n) {  // layout, q k v o lse, q_row_start, scale, stream
  s2_tensors t;
  float scale;
  void *layout, *stream;
  int32_t row0;
  int64_t ksize[3];
  if (!count_is(n, 9) || !tensors_of(a + 1, 5, t) || !sizes_of(a[2], -1, ksize, 3) || !as_address(a[0], layout) || !as_i32(a[6], row0) ||
      !as_float(a[7], scale) || !as_address(a[8], stream))
    return nullptr;
  const int32_t rows = t.seqlen;
  t.seqlen = (int32_t)ksize[2];
  return status_of([&] { return api.f.fwd_rows(static_cast<s2_layout*>(layout), &t, row0, rows, scale, stream); });
}

PyObject* fwd_varlen(PyObject*, PyObject* const* a, Py_ssize_t n) {  // layout, q k v o lse, cu_seqlens, max_seqlen, scale, stream
  s2_tensors t;
  float scale;
  void *layout, *stream;
  const int32_t* cu;
  int32_t seqs, longest;
  if (!count_is(n, 10) || !tensors_of(a + 1, 5, t) || !offsets_of(a[6], a[1], cu, seqs) || !as_address(a[0], layout) || !as_i32(a[7], longest) ||
      !as_float(a[8], scale) || !as_address(a[9], stream))
    return nullptr;
  return status_of([&] { return api.f.fwd_varlen(static_cast<s2_layout*>(layout), &t, cu, seqs, longest, scale, stream); });
}

PyObject* bwd_stages(PyObject*, PyObject* const* a, Py_ssize_t n) {  // layout, nine tensors, scale, workspace, stages, stream
  s2_tensors t;
  float scale;
  void *layout, *stream, *ws;
  size_t bytes;
  int32_t stages;
  if (!count_is(n, 14) || !tensors_of(a + 1, 9, t) || !as_address(a[0], layout) || !as_float(a[10], scale) || !workspace_of(a[11], ws, bytes) ||
      !as_i32(a[12], stages) || !as_address(a[13], stream))
    return nullptr;
  return status_of([&] { return api.f.bwd_stages(static_cast<s2_layout*>(layout), &t, scale, ws, bytes, stages, stream); });
}

PyObject* bwd_varlen(PyObject*, PyObject* const* a, Py_ssize_t n) {  // layout, nine tensors, cu_seqlens, max_seqlen, scale, workspace, stream
  s2_tensors t;
  float scale;
  void *layout, *stream, *ws;
  size_t bytes;
  const int32_t* cu;
  int32_t seqs, longest;
  if (!count_is(n, 15) || !tensors_of(a + 1, 9, t) || !offsets_of(a[10], a[1], cu, seqs) || !as_address(a[0], layout) || !as_i32(a[11], longest) ||
      !as_float(a[12], scale) || !workspace_of(a[13], ws, bytes) || !as_address(a[14], stream))
    return nullptr;
  return status_of([&] { return api.f.bwd_varlen(static_cast<s2_layout*>(layout), &t, cu, seqs, longest, scale, ws, bytes, stream); });
}

PyObject* dense_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {  // q k v o lse, scale, stream
  s2_tensors t;
  float scale;
  void* stream;
  if (!count_is(n, 7) || !tensors_of(a, 5, t) || !as_float(a[5], scale) || !as_address(a[6], stream)) return nullptr;
  return status_of([&] { return api.f.dense_fwd(&t, scale, stream); });
}

PyObject* dense_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {  // nine tensors, scale, workspace, stream
  s2_tensors t;
  float scale;
  void *stream, *ws;
  size_t bytes;
  if (!count_is(n, 12) || !tensors_of(a, 9, t) || !as_float(a[9], scale) || !workspace_of(a[10], ws, bytes) || !as_address(a[11], stream)) return nullptr;
  return status_of([&] { return api.f.dense_bwd(&t, scale, ws, bytes, stream); });
}

// q, caches, seq_lens, o, lse, max_len, num_splits
bool decode_of(PyObject* const* a, PyObject* max_len, PyObject* splits, s2_decode_args& d) {
  int64_t size[3];
  if (!sizes_of(a[0], 3, size) || !contiguous(a[0]) || !contiguous(a[4])) return false;
  const Ref ks(strides_of(a[1])), vs(ks.o ? strides_of(a[2]) : nullptr);
  if (!vs.o || !same(ks.o, vs.o) || !unit_stride(ks.o, 3)) return false;
  if (!data_of(a[0], d.q) || !data_of(a[1], d.k_cache) || !data_of(a[2], d.v_cache) || !data_of(a[3], d.seq_lens) || !data_of(a[4], d.o) ||
      !data_of(a[5], d.lse))
    return false;
  d.nseq = (int32_t)size[0];
  d.heads = (int32_t)size[1];
  d.head_dim = (int32_t)size[2];
  return as_i32(max_len, d.max_len) && as_i32(splits, d.num_splits) && stride_at(ks.o, 0, d.kv_stride_seq) && stride_at(ks.o, 1, d.kv_stride_head) &&
         stride_at(ks.o, 2, d.kv_stride_tok);
}

// params or layout, q k v seq_lens o lse, scale, workspace, max_len, num_splits, stream
template <bool LAYOUT>
PyObject* decode_workspace(PyObject* const* a, Py_ssize_t n) {
  s2_decode_args d;
  float scale;
  void *pattern, *stream, *ws;
  size_t bytes;
  if (!count_is(n, 12) || !decode_of(a + 1, a[9], a[10], d) || !as_address(a[0], pattern) || !as_float(a[7], scale) || !workspace_of(a[8], ws, bytes) ||
      !as_address(a[11], stream))
    return nullptr;
  return status_of([&] {
    if constexpr (LAYOUT)
      return api.f.decode_layout(static_cast<s2_layout*>(pattern), &d, scale, ws, bytes, stream);
    else
      return api.f.decode(static_cast<s2_layout_params*>(pattern), &d, scale, ws, bytes, stream);
  });
}
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) { return decode_workspace<false>(a, n); }
PyObject* decode_layout(PyObject*, PyObject* const* a, Py_ssize_t n) { return decode_workspace<true>(a, n); }

PyObject* decode_static(PyObject*, PyObject* const* a, Py_ssize_t n) {  // params, q k v seq_lens o lse, scale, max_len, num_splits, stream
  s2_decode_args d;
  float scale;
  void *params, *stream;
  if (!count_is(n, 11) || !decode_of(a + 1, a[8], a[9], d) || !as_address(a[0], params) || !as_float(a[7], scale) || !as_address(a[10], stream)) return nullptr;
  return status_of([&] { return api.f.decode_static(static_cast<s2_layout_params*>(params), &d, scale, stream); });
}

// params or layout, q k v block_table seq_lens o lse, scale, workspace, missing, num_splits, stream
template <bool LAYOUT>
PyObject* paged(PyObject* const* a, Py_ssize_t n) {
  s2_paged_decode_args d;
  float scale;
  void *pattern, *stream, *ws;
  size_t bytes;
  int64_t size[3], table[3], pages;
  if (!count_is(n, 13) || !sizes_of(a[1], 3, size) || !contiguous(a[1]) || !contiguous(a[6]) || !contiguous(a[4])) return nullptr;
  const Ref ks(strides_of(a[2])), vs(ks.o ? strides_of(a[3]) : nullptr);
  if (!vs.o || !same(ks.o, vs.o) || !unit_stride(ks.o, 2)) return nullptr;
  if (!sizes_of(a[4], -1, table, 2)) {
    // (a table of fewer than two sizes is not [nseq, heads, ...])
    if (PyErr_ExceptionMatches(PyExc_IndexError)) PyErr_SetNone(PyExc_AssertionError);
    return nullptr;
  }
  if (table[0] != size[0] || table[1] != size[1]) {
    fail_assert();
    return nullptr;
  }
  if (!sizes_of(a[4], -1, table, 3) || !sizes_of(a[2], -1, &pages, 1)) return nullptr;
  if (!data_of(a[1], d.q) || !data_of(a[2], d.k_pages) || !data_of(a[3], d.v_pages) || !data_of(a[4], d.block_table) || !data_of(a[5], d.seq_lens) ||
      !data_of(a[6], d.o) || !data_of(a[7], d.lse) || !data_of(a[10], d.missing))
    return nullptr;
  d.nseq = (int32_t)size[0];
  d.heads = (int32_t)size[1];
  d.head_dim = (int32_t)size[2];
  d.max_blocks = (int32_t)table[2];
  d.num_pages = (int32_t)pages;
  if (!as_i32(a[11], d.num_splits) || !stride_at(ks.o, 0, d.page_stride) || !stride_at(ks.o, 1, d.tok_stride)) return nullptr;
  if (!as_address(a[0], pattern) || !as_float(a[8], scale) || !workspace_of(a[9], ws, bytes) || !as_address(a[12], stream)) return nullptr;
  return status_of([&] {
    if constexpr (LAYOUT)
      return api.f.decode_paged_layout(static_cast<s2_layout*>(pattern), &d, scale, ws, bytes, stream);
    else
      return api.f.decode_paged(static_cast<s2_layout_params*>(pattern), &d, scale, ws, bytes, stream);
  });
}
PyObject* decode_paged(PyObject*, PyObject* const* a, Py_ssize_t n) { return paged<false>(a, n); }
PyObject* decode_paged_layout(PyObject*, PyObject* const* a, Py_ssize_t n) { return paged<true>(a, n); }

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!count_is(n, kEntryPoints)) return nullptr;
  void* at[kEntryPoints];
  for (Py_ssize_t i = 0; i < n; ++i) {
    at[i] = PyLong_AsVoidPtr(a[i]);
    if (!at[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address");
      return nullptr;
    }
  }
  for (Py_ssize_t i = 0; i < n; ++i) api.at[i] = at[i];
  Py_RETURN_NONE;
}

#define S2_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {S2_METHOD(bind),          S2_METHOD(fwd),          S2_METHOD(fwd_rows),      S2_METHOD(fwd_varlen),
                         S2_METHOD(bwd_stages),    S2_METHOD(bwd_varlen),   S2_METHOD(dense_fwd),     S2_METHOD(dense_bwd),
                         S2_METHOD(decode),        S2_METHOD(decode_static), S2_METHOD(decode_layout), S2_METHOD(decode_paged),
                         S2_METHOD(decode_paged_layout), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  struct {
    PyObject** at;
    const char* text;
  } const all[] = {{&names.data_ptr, "data_ptr"}, {&names.stride, "stride"},   {&names.shape, "shape"}, {&names.is_contiguous, "is_contiguous"},
                   {&names.numel, "numel"},       {&names.element_size, "element_size"}, {&names.value, "value"}};
  for (const auto& n : all)
    if (!(*n.at = PyUnicode_InternFromString(n.text))) return nullptr;
  const Ref m(PyModule_Create(&module));
  if (!m.o) return nullptr;
#define X(entry, name) #entry,
  const char* const entries[] = {S2_ENTRY_POINTS(X)};
#undef X
  const Ref order(PyTuple_New(kEntryPoints));
  if (!order.o) return nullptr;
  for (Py_ssize_t i = 0; i < kEntryPoints; ++i) {
    PyObject* const name = PyUnicode_FromString(entries[i]);
    if (!name) return nullptr;
    PyTuple_SET_ITEM(order.o, i, name);
  }
  if (PyObject_SetAttrString(m.o, "entry_points", order.o)) return nullptr;
  Py_INCREF(m.o);
  return m.o;
}
