// Marshalling of the calls a decoding loop makes, for binding.py: tensors to device pointers, strides
// and the current stream, then the C ABI.  A call is one or two kernels of a few microseconds, and a loop of
// such calls is bound by the host: through ctypes a layer took 5.7 us of host time, 2.5 of them
// the launch; a foreign-function conversion per argument and a Python-level call per pointer
// were most of the rest.  Host code only; links nothing but Python (the library's functions are
// handed over as addresses).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>
#include <string.h>

#include "talon.h"

namespace {

// ---- the C ABI, as loaded by binding.py
struct Abi {
  decltype(&talon_last_error_string) last_error_string;
  decltype(&talon_tree_init) tree_init;
  decltype(&talon_expand_layer) expand_layer;
  decltype(&talon_select_budget) select_budget;
  decltype(&talon_expand_select_layer) expand_select_layer;
  decltype(&talon_expand_tree) expand_tree;
  decltype(&talon_build_tree) build_tree;
  decltype(&talon_build_tree_ahead) build_tree_ahead;
  decltype(&talon_expand_literal) expand_literal;
  decltype(&talon_expand_literal_ahead) expand_literal_ahead;
  decltype(&talon_target_argmax) target_argmax;
  decltype(&talon_greedy_accept) greedy_accept;
  decltype(&talon_compact_kv) compact_kv;
  decltype(&talon_build_tree_mask) build_tree_mask;
  decltype(&talon_tree_attention) tree_attention;
  decltype(&talon_tree_attention_static) tree_attention_static;
};
constexpr int kFunctions = sizeof(Abi) / sizeof(void*);
Abi g_abi;   // (set under the interpreter lock)

// ---- objects of Python handed over once
PyObject *g_error, *g_float32, *g_bfloat16, *g_int_of, *g_float_of, *g_stream_of, *g_raw_stream, *g_device,
    *g_initialized;   // (the last three may be None)
// ---- interned names
PyObject *n_data_ptr, *n_stride, *n_shape, *n_dtype, *n_nbytes, *n_token, *n_logit, *n_prob, *n_edge_logp, *n_row_max, *n_row_lse,
    *n_is_contiguous, *n_numel;

// One call: the first failure is kept (Python's error indicator is set), later steps do nothing.
struct Call {
  bool ok = true;
  Py_buffer state = {};   // the tree state's C struct
  bool have_state = false;

  ~Call() { if (have_state) PyBuffer_Release(&state); }

  void fail() { ok = false; }
  void refuse(int code, const char* message) {
    if (!ok) return;
    ok = false;
    PyObject* e = PyObject_CallFunction(g_error, "is", code, message);
    if (e) { PyErr_SetObject(g_error, e); Py_DECREF(e); }
  }
  PyObject* attr(PyObject* o, PyObject* name) {   // new reference
    if (!ok) return nullptr;
    PyObject* r = PyObject_GetAttr(o, name);
    if (!r) ok = false;
    return r;
  }
  PyObject* call(PyObject* o, PyObject* name) {   // new reference
    if (!ok) return nullptr;
    PyObject* r = PyObject_CallMethodNoArgs(o, name);
    if (!r) ok = false;
    return r;
  }
  long long integer_of(PyObject* o) {   // of a Python int
    if (!ok) return 0;
    if (!PyLong_Check(o)) {
      PyErr_Format(PyExc_TypeError, "an integer is required, not %.100s", Py_TYPE(o)->tp_name);
      ok = false;
      return 0;
    }
    return static_cast<long long>(PyLong_AsUnsignedLongLongMask(o));
  }
  // A caller's numbers: Python's own at once, others (numpy's, tensors of one element, ctypes', ...) as a
  // foreign function takes them.
  int32_t i32(PyObject* o) {
    if (!ok || PyLong_Check(o)) return static_cast<int32_t>(integer_of(o));
    PyObject* v = PyObject_CallOneArg(g_int_of, o);
    if (!v) ok = false;
    return static_cast<int32_t>(steal_i64(v));
  }
  float f32(PyObject* o) {
    if (!ok) return 0.f;
    const bool own = PyFloat_Check(o) || PyLong_Check(o);
    PyObject* v = own ? o : PyObject_CallOneArg(g_float_of, o);
    const double d = v ? PyFloat_AsDouble(v) : -1.0;
    if (d == -1.0 && PyErr_Occurred()) ok = false;
    if (!own) Py_XDECREF(v);
    return static_cast<float>(d);
  }
  int64_t steal_i64(PyObject* o) {
    const int64_t v = o ? integer_of(o) : 0;
    Py_XDECREF(o);
    return v;
  }
  // device address of a tensor, or NULL for None
  void* ptr(PyObject* t) {
    if (!ok || t == Py_None) return nullptr;
    PyObject* r = call(t, n_data_ptr);
    void* p = nullptr;
    if (r) {
      p = PyLong_AsVoidPtr(r);
      if (!p && PyErr_Occurred()) ok = false;
      Py_DECREF(r);
    }
    return p;
  }
  void* ptr_attr(PyObject* o, PyObject* name) {
    PyObject* t = attr(o, name);
    void* p = t ? ptr(t) : nullptr;
    Py_XDECREF(t);
    return p;
  }
  size_t nbytes(PyObject* t) { return static_cast<size_t>(steal_i64(attr(t, n_nbytes))); }
  // the ctypes struct that names the tree state's buffers
  const talon_tree_state* tree(PyObject* c) {
    if (!ok) return nullptr;
    if (PyObject_GetBuffer(c, &state, PyBUF_SIMPLE) != 0) { ok = false; return nullptr; }
    have_state = true;
    if (state.len != static_cast<Py_ssize_t>(sizeof(talon_tree_state))) {
      PyErr_SetString(PyExc_TypeError, "the tree state's C struct is required");
      ok = false;
      return nullptr;
    }
    return static_cast<const talon_tree_state*>(state.buf);
  }
  // the current stream (None), an object with a cuda_stream, or a raw handle
  void* stream(PyObject* s) {
    if (!ok) return nullptr;
    PyObject* r = nullptr;
    if (s == Py_None && g_raw_stream != Py_None && g_device != Py_None) {   // as binding._stream does it
      PyObject* yes = PyObject_CallNoArgs(g_initialized);
      if (yes == Py_True) {
        PyObject* device = PyObject_CallNoArgs(g_device);
        r = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
        Py_XDECREF(device);
      }
      Py_XDECREF(yes);
      if (!r && PyErr_Occurred()) { ok = false; return nullptr; }
    }
    if (!r) r = PyObject_CallOneArg(g_stream_of, s);
    if (!r) { ok = false; return nullptr; }
    void* p = PyLong_AsVoidPtr(r);
    if (!p && PyErr_Occurred()) ok = false;
    Py_DECREF(r);
    return p;
  }
  int64_t item(PyObject* tuple, Py_ssize_t i) { return ok ? integer_of(PyTuple_GET_ITEM(tuple, i)) : 0; }
  // A tuple of n items (or more, where asked for), new reference.
  PyObject* tuple_of(PyObject* t, Py_ssize_t n, const char* message, bool method, PyObject* name, bool or_more = false) {
    PyObject* r = method ? call(t, name) : attr(t, name);
    if (r && (!PyTuple_Check(r) || PyTuple_GET_SIZE(r) < n || (PyTuple_GET_SIZE(r) > n && !or_more))) {
      Py_DECREF(r);
      r = nullptr;
      refuse(TALON_ERR_INVALID_ARG, message);
    }
    return r;
  }
  void contiguous(PyObject* t, const char* message) {
    PyObject* r = call(t, n_is_contiguous);
    if (r && r != Py_True) refuse(TALON_ERR_INVALID_ARG, message);
    Py_XDECREF(r);
  }
};

// [B][rows][V] logits with contiguous rows
struct Logits {
  void* p = nullptr;
  int dtype = 0;
  int64_t row_stride = 0, seq_stride = 0, sequences = 0, rows = 0;
  int32_t vocab = 0;
  int64_t width = 0;
  Logits(Call& c, PyObject* t, PyObject* vocab_arg) {
    PyObject* dt = c.attr(t, n_dtype);
    if (dt == g_float32) dtype = TALON_DTYPE_F32;
    else if (dt == g_bfloat16) dtype = TALON_DTYPE_BF16;
    else if (dt) {
      PyObject* text = PyUnicode_FromFormat("logits dtype %S", dt);
      if (text) { c.refuse(TALON_ERR_UNSUPPORTED, PyUnicode_AsUTF8(text)); Py_DECREF(text); } else c.fail();
    }
    Py_XDECREF(dt);
    const char* shape_text = "logits must be [B][rows][V] with contiguous rows";
    PyObject* strides = c.tuple_of(t, 3, shape_text, true, n_stride);
    if (strides) {
      seq_stride = c.item(strides, 0);
      row_stride = c.item(strides, 1);
      if (c.item(strides, 2) != 1) c.refuse(TALON_ERR_INVALID_ARG, shape_text);
      Py_DECREF(strides);
    }
    PyObject* shape = c.tuple_of(t, 3, shape_text, false, n_shape);
    if (shape) {
      sequences = c.item(shape, 0);
      rows = c.item(shape, 1);
      width = c.item(shape, 2);
      Py_DECREF(shape);
    }
    vocab = vocab_arg == Py_None ? static_cast<int32_t>(width) : c.i32(vocab_arg);
    p = c.ptr(t);
  }
  // every row of the tensor may be read: rows by node id, the vocabulary inside the tensor
  bool all_rows(const talon_tree_state* st, int row_mode) const {
    return row_mode == TALON_ROWS_BY_NODE && vocab <= width && sequences >= st->B && rows > 0;
  }
};

struct Outputs {   // binding.Candidates
  int32_t* token;
  float *logit, *prob;
  double* edge_logp;
  float* row_max;
  double* row_lse;
  Outputs(Call& c, PyObject* o)
      : token(static_cast<int32_t*>(c.ptr_attr(o, n_token))), logit(static_cast<float*>(c.ptr_attr(o, n_logit))),
        prob(static_cast<float*>(c.ptr_attr(o, n_prob))), edge_logp(static_cast<double*>(c.ptr_attr(o, n_edge_logp))),
        row_max(static_cast<float*>(c.ptr_attr(o, n_row_max))), row_lse(static_cast<double*>(c.ptr_attr(o, n_row_lse))) {}
};

PyObject* result(Call& c, int rc) {
  if (c.ok && rc != TALON_OK) c.refuse(rc, g_abi.last_error_string());
  if (!c.ok) return nullptr;
  Py_RETURN_NONE;
}

bool arguments(Py_ssize_t got, Py_ssize_t want) {
  if (got == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, got);
  return false;
}

#define RUN(rc, expression)                                  \
  int rc = TALON_OK;                                         \
  if (c.ok) {                                                \
    Py_BEGIN_ALLOW_THREADS rc = (expression);                \
    Py_END_ALLOW_THREADS                                     \
  }

// (st, root_token, stream)
PyObject* tree_init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 3)) return nullptr;
  Call c;
  const talon_tree_state* st = c.tree(a[0]);
  const int32_t* root = static_cast<const int32_t*>(c.ptr(a[1]));
  void* s = c.stream(a[2]);
  RUN(rc, g_abi.tree_init(st, root, s))
  return result(c, rc);
}

// (logits, st, k, cand, workspace, row_mode, layer, vocab, stream)
PyObject* expand_layer(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 9)) return nullptr;
  Call c;
  const Logits l(c, a[0], a[7]);
  const talon_tree_state* st = c.tree(a[1]);
  const int32_t k = c.i32(a[2]);
  const Outputs o(c, a[3]);
  void* ws = c.ptr(a[4]);
  const size_t bytes = c.nbytes(a[4]);
  const int mode = c.i32(a[5]), layer = c.i32(a[6]);
  void* s = c.stream(a[8]);
  RUN(rc, g_abi.expand_layer(l.p, l.dtype, l.row_stride, l.seq_stride, mode, layer, st, l.vocab, k, o.token, o.logit, o.prob, o.edge_logp,
                             o.row_max, o.row_lse, ws, bytes, s))
  return result(c, rc);
}

// (st, k, cand, mu, K_init, init_layers, max_depth, stream)
PyObject* select_budget(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 8)) return nullptr;
  Call c;
  const talon_tree_state* st = c.tree(a[0]);
  const int32_t k = c.i32(a[1]);
  const int32_t* token = static_cast<const int32_t*>(c.ptr_attr(a[2], n_token));
  const float* prob = static_cast<const float*>(c.ptr_attr(a[2], n_prob));
  const double* edge = static_cast<const double*>(c.ptr_attr(a[2], n_edge_logp));
  const float mu = c.f32(a[3]);
  const int32_t K_init = c.i32(a[4]), init_layers = c.i32(a[5]), max_depth = c.i32(a[6]);
  void* s = c.stream(a[7]);
  RUN(rc, g_abi.select_budget(st, k, token, prob, edge, mu, K_init, init_layers, max_depth, s))
  return result(c, rc);
}

// (logits, st, k, mu, K_init, init_layers, max_depth, cand, workspace, layer, row_mode, vocab, stream); the layer
// has no effect on talon_expand_tree
template <bool ONE>
PyObject* expand_select(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 13)) return nullptr;
  Call c;
  const Logits l(c, a[0], a[11]);
  const talon_tree_state* st = c.tree(a[1]);
  const int32_t k = c.i32(a[2]);
  const float mu = c.f32(a[3]);
  const int32_t K_init = c.i32(a[4]), init_layers = c.i32(a[5]), max_depth = c.i32(a[6]);
  const Outputs o(c, a[7]);
  void* ws = c.ptr(a[8]);
  const size_t bytes = c.nbytes(a[8]);
  const int layer = c.i32(a[9]), mode = c.i32(a[10]);
  void* s = c.stream(a[12]);
  RUN(rc, ONE ? g_abi.expand_select_layer(l.p, l.dtype, l.row_stride, l.seq_stride, mode, layer, st, l.vocab, k, mu, K_init, init_layers,
                                          max_depth, o.token, o.logit, o.prob, o.edge_logp, o.row_max, o.row_lse, ws, bytes, s)
              : g_abi.expand_tree(l.p, l.dtype, l.row_stride, l.seq_stride, mode, st, l.vocab, k, mu, K_init, init_layers, max_depth,
                                  o.token, o.logit, o.prob, o.edge_logp, o.row_max, o.row_lse, ws, bytes, s))
  return result(c, rc);
}

// (root_token, logits, st, k, mu, K_init, init_layers, max_depth, cand, workspace, mask, row_mode, vocab, stream)
PyObject* build_tree(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 14)) return nullptr;
  Call c;
  const int32_t* root = static_cast<const int32_t*>(c.ptr(a[0]));
  const Logits l(c, a[1], a[12]);
  const talon_tree_state* st = c.tree(a[2]);
  const int32_t k = c.i32(a[3]);
  const float mu = c.f32(a[4]);
  const int32_t K_init = c.i32(a[5]), init_layers = c.i32(a[6]), max_depth = c.i32(a[7]);
  const Outputs o(c, a[8]);
  void* ws = c.ptr(a[9]);
  const size_t bytes = c.nbytes(a[9]);
  uint64_t* mask = static_cast<uint64_t*>(c.ptr(a[10]));
  const int mode = c.i32(a[11]);
  void* s = c.stream(a[13]);
  RUN(rc, l.all_rows(st, mode)
              ? g_abi.build_tree_ahead(root, l.p, l.dtype, l.row_stride, l.seq_stride, static_cast<int32_t>(l.rows), st, l.vocab, k, mu,
                                       K_init, init_layers, max_depth, o.token, o.logit, o.prob, o.edge_logp, o.row_max, o.row_lse, mask, ws, bytes, s)
              : g_abi.build_tree(root, l.p, l.dtype, l.row_stride, l.seq_stride, mode, st, l.vocab, k, mu, K_init, init_layers, max_depth,
                                 o.token, o.logit, o.prob, o.edge_logp, o.row_max, o.row_lse, mask, ws, bytes, s))
  return result(c, rc);
}

// (logits, st, layers, mu, K_init, init_layers, max_depth, workspace, row_mode, vocab, stream)
PyObject* expand_literal(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 11)) return nullptr;
  Call c;
  const Logits l(c, a[0], a[9]);
  const talon_tree_state* st = c.tree(a[1]);
  const int32_t layers = c.i32(a[2]);
  const float mu = c.f32(a[3]);
  const int32_t K_init = c.i32(a[4]), init_layers = c.i32(a[5]), max_depth = c.i32(a[6]);
  void* ws = c.ptr(a[7]);
  const size_t bytes = c.nbytes(a[7]);
  const int mode = c.i32(a[8]);
  void* s = c.stream(a[10]);
  RUN(rc, l.all_rows(st, mode) ? g_abi.expand_literal_ahead(l.p, l.dtype, l.row_stride, l.seq_stride, static_cast<int32_t>(l.rows), layers,
                                                            st, l.vocab, mu, K_init, init_layers, max_depth, ws, bytes, s)
                               : g_abi.expand_literal(l.p, l.dtype, l.row_stride, l.seq_stride, mode, layers, st, l.vocab, mu, K_init,
                                                      init_layers, max_depth, ws, bytes, s))
  return result(c, rc);
}

// (logits, st, target_token, target_prob, scan_status, workspace, vocab, stream)
PyObject* target_argmax(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 8)) return nullptr;
  Call c;
  const Logits l(c, a[0], a[6]);
  const talon_tree_state* st = c.tree(a[1]);
  int32_t* token = static_cast<int32_t*>(c.ptr(a[2]));
  float* prob = static_cast<float*>(c.ptr(a[3]));
  uint32_t* status = static_cast<uint32_t*>(c.ptr(a[4]));
  void* ws = c.ptr(a[5]);
  const size_t bytes = c.nbytes(a[5]);
  void* s = c.stream(a[7]);
  RUN(rc, g_abi.target_argmax(l.p, l.dtype, l.row_stride, l.seq_stride, st, l.vocab, token, prob, status, ws, bytes, s))
  return result(c, rc);
}

// (st, target_token, scan_status, path, accept_len, bonus_token, stream)
PyObject* greedy_accept(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 7)) return nullptr;
  Call c;
  const talon_tree_state* st = c.tree(a[0]);
  const int32_t* target = static_cast<const int32_t*>(c.ptr(a[1]));
  const uint32_t* status = static_cast<const uint32_t*>(c.ptr(a[2]));
  int32_t *path = static_cast<int32_t*>(c.ptr(a[3])), *len = static_cast<int32_t*>(c.ptr(a[4])), *bonus = static_cast<int32_t*>(c.ptr(a[5]));
  void* s = c.stream(a[6]);
  RUN(rc, g_abi.greedy_accept(st, target, status, path, len, bonus, s))
  return result(c, rc);
}

// Strides of a [B][L][Hkv][Dh] view that both prefix tensors share; *shape1 (optional): its L.
void prefix_strides(Call& c, PyObject* k, PyObject* v, int64_t* b, int64_t* t, int64_t* h, int64_t* shape1) {
  const char* text = "k_prefix and v_prefix must share strides, Dh contiguous";
  PyObject* ks = c.tuple_of(k, 4, text, true, n_stride);
  PyObject* vs = c.tuple_of(v, 4, text, true, n_stride);
  if (ks && vs) {
    const int same = PyObject_RichCompareBool(ks, vs, Py_EQ);
    if (same < 0) c.fail();
    else if (!same || c.item(ks, 3) != 1) c.refuse(TALON_ERR_INVALID_ARG, text);
    *b = c.item(ks, 0);
    *t = c.item(ks, 1);
    *h = c.item(ks, 2);
  }
  Py_XDECREF(ks);
  Py_XDECREF(vs);
  if (shape1) {
    PyObject* shape = c.tuple_of(k, 4, text, false, n_shape);
    if (shape) *shape1 = c.item(shape, 1);
    Py_XDECREF(shape);
  }
}

struct Shape4 {
  int32_t d[4] = {0, 0, 0, 0};
  Shape4(Call& c, PyObject* t, const char* text) {
    PyObject* shape = c.tuple_of(t, 4, text, false, n_shape);
    for (int i = 0; shape && i < 4; ++i) d[i] = static_cast<int32_t>(c.item(shape, i));
    Py_XDECREF(shape);
  }
};

// (k_tree, v_tree, path, accept_len, prefix_len, new_prefix_len, k_prefix, v_prefix, stream)
PyObject* compact_kv(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 9)) return nullptr;
  Call c;
  const Shape4 kt(c, a[0], "k_tree must be [B][N_pad][Hkv][Dh]");
  int64_t sb = 0, st = 0, sh = 0, capacity = 0;
  prefix_strides(c, a[6], a[7], &sb, &st, &sh, &capacity);
  void *k_tree = c.ptr(a[0]), *v_tree = c.ptr(a[1]);
  const int32_t *path = static_cast<const int32_t*>(c.ptr(a[2])), *len = static_cast<const int32_t*>(c.ptr(a[3])),
                *prefix = static_cast<const int32_t*>(c.ptr(a[4]));
  int32_t* new_prefix = static_cast<int32_t*>(c.ptr(a[5]));
  void *k_prefix = c.ptr(a[6]), *v_prefix = c.ptr(a[7]);
  void* s = c.stream(a[8]);
  RUN(rc, g_abi.compact_kv(k_tree, v_tree, path, len, prefix, new_prefix, k_prefix, v_prefix, kt.d[0], kt.d[1], kt.d[2], kt.d[3],
                           static_cast<int32_t>(capacity), sb, st, sh, s))
  return result(c, rc);
}

// (st, mask, stream)
PyObject* build_tree_mask(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 3)) return nullptr;
  Call c;
  const talon_tree_state* st = c.tree(a[0]);
  uint64_t* mask = static_cast<uint64_t*>(c.ptr(a[1]));
  void* s = c.stream(a[2]);
  RUN(rc, g_abi.build_tree_mask(st, mask, s))
  return result(c, rc);
}

// (q, k_prefix, v_prefix, k_tree, v_tree, mask, n_nodes, prefix_len, max_prefix_len, out, out_lse, workspace, scale, stream, static)
PyObject* tree_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 15)) return nullptr;
  Call c;
  const Shape4 q(c, a[0], "q must be [B][N_pad][Hq][Dh]");
  int32_t Hkv = 0;
  PyObject* kt = c.tuple_of(a[3], 3, "k_tree must be [B][N_pad][Hkv][Dh]", false, n_shape, true);   // (Dh is q's)
  if (kt) Hkv = static_cast<int32_t>(c.item(kt, 2));
  Py_XDECREF(kt);
  const char* text = "q, k_tree, v_tree, mask and out must be contiguous";
  PyObject* const dense[] = {a[0], a[3], a[4], a[9], a[5]};
  for (PyObject* t : dense) c.contiguous(t, text);
  const int32_t most = c.i32(a[8]);
  bool prefix = most != 0 && a[1] != Py_None;
  if (prefix) prefix = c.steal_i64(c.call(a[1], n_numel)) != 0;   // an empty one: the tree attends to itself only
  int64_t sb = q.d[3], st = q.d[3], sh = q.d[3];
  if (prefix) prefix_strides(c, a[1], a[2], &sb, &st, &sh, nullptr);
  void *qp = c.ptr(a[0]), *kp = prefix ? c.ptr(a[1]) : nullptr, *vp = prefix ? c.ptr(a[2]) : nullptr, *ktp = c.ptr(a[3]), *vtp = c.ptr(a[4]);
  const uint64_t* mask = static_cast<const uint64_t*>(c.ptr(a[5]));
  const int32_t *nodes = static_cast<const int32_t*>(c.ptr(a[6])), *len = static_cast<const int32_t*>(c.ptr(a[7]));
  void* out = c.ptr(a[9]);
  float* lse = static_cast<float*>(c.ptr(a[10]));
  void* ws = c.ptr(a[11]);
  const size_t bytes = a[11] == Py_None ? 0 : c.nbytes(a[11]);
  const float scale = c.f32(a[12]);
  void* s = c.stream(a[13]);
  const int own = PyObject_IsTrue(a[14]);
  if (own < 0) c.fail();
  RUN(rc, own ? g_abi.tree_attention_static(qp, kp, vp, ktp, vtp, mask, nodes, len, q.d[0], q.d[1], q.d[2], Hkv, q.d[3], most, sb, st, sh,
                                            scale, out, lse, s)
              : g_abi.tree_attention(qp, kp, vp, ktp, vtp, mask, nodes, len, q.d[0], q.d[1], q.d[2], Hkv, q.d[3], most, sb, st, sh, scale,
                                     out, lse, ws, bytes, s))
  return result(c, rc);
}

// (addresses of the functions in the order of Abi, TalonError, torch.float32, torch.bfloat16, binding._int_of and _float_of,
// binding._stream and what it asks: raw handle of a device's current stream, current device, is the GPU initialised)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!arguments(n, 10)) return nullptr;
  if (!PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != kFunctions) {
    PyErr_Format(PyExc_TypeError, "%d addresses expected", kFunctions);
    return nullptr;
  }
  void* p[kFunctions];
  for (int i = 0; i < kFunctions; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[0], i));
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a function's address is NULL");
      return nullptr;
    }
  }
  static_assert(sizeof(g_abi) == sizeof(p), "function pointers only");
  memcpy(&g_abi, p, sizeof(p));
  PyObject** const keep[] = {&g_error, &g_float32, &g_bfloat16, &g_int_of, &g_float_of, &g_stream_of, &g_raw_stream, &g_device, &g_initialized};
  for (int i = 0; i < 9; ++i) {
    Py_INCREF(a[1 + i]);
    Py_XDECREF(*keep[i]);
    *keep[i] = a[1 + i];
  }
  Py_RETURN_NONE;
}

#define METHOD(name, f) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {METHOD(bind, bind), METHOD(tree_init, tree_init), METHOD(expand_layer, expand_layer),
                           METHOD(select_budget, select_budget), METHOD(expand_select_layer, expand_select<true>),
                           METHOD(expand_tree, expand_select<false>), METHOD(build_tree, build_tree),
                           METHOD(expand_literal, expand_literal), METHOD(target_argmax, target_argmax),
                           METHOD(greedy_accept, greedy_accept), METHOD(compact_kv, compact_kv),
                           METHOD(build_tree_mask, build_tree_mask), METHOD(tree_attention, tree_attention),
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_talon_marshal", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__talon_marshal(void) {
  struct { PyObject** at; const char* text; } const names[] = {
      {&n_data_ptr, "data_ptr"}, {&n_stride, "stride"}, {&n_shape, "shape"}, {&n_dtype, "dtype"}, {&n_nbytes, "nbytes"},
      {&n_token, "token"}, {&n_logit, "logit"}, {&n_prob, "prob"}, {&n_edge_logp, "edge_logp"}, {&n_row_max, "row_max"},
      {&n_row_lse, "row_lse"}, {&n_is_contiguous, "is_contiguous"}, {&n_numel, "numel"}};
  for (const auto& n : names)
    if (!(*n.at = PyUnicode_InternFromString(n.text))) return nullptr;
  return PyModule_Create(&g_module);
}
