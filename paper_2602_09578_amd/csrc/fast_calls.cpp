// The Python binding's short way into the library for the calls of a decode loop: the same checks of types,
// extents, device and contiguity as in binding.py, made on the tensors themselves, and the call, in one step.
// A call whose arguments are not plainly right is not made here: None is returned and the binding goes its long
// way, which reports what is wrong.  (Host time of a call, long way and short: attention of 16 sequences 7.9 and 3.5 us,
// log-probabilities 5.8 and 3.0, prompt scatter 7.4 and 3.5; most of what is left is the launch.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <exception>
#include <initializer_list>

#include "marl_decode.h"

namespace {

PyObject* g_stream_of = nullptr;      // device index -> the current stream's handle
PyObject* g_attn_shape = nullptr;     // the ctypes structures' types
PyObject* g_prefill_shape = nullptr;
decltype(&marl_decode_attn) f_decode_attn;
decltype(&marl_token_logprobs) f_token_logprobs;
decltype(&marl_kv_append) f_kv_append;
decltype(&marl_sample_tokens) f_sample_tokens;
decltype(&marl_sample_tokens_top_p) f_sample_tokens_top_p;
decltype(&marl_prefill_attn) f_prefill_attn;
decltype(&marl_kv_write_prompt) f_kv_write_prompt;

struct Call {
  bool ok = true;
  int device = -1;   // of the first tensor

  // The data of a plain, contiguous device tensor of the given type and sizes (-1: any, at least that many dimensions are
  // there); null for None.
  const at::Tensor* tensor(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> sizes) {
    if (!ok || !THPVariable_CheckExact(o)) return fail();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous() || t.dim() != (int64_t)sizes.size()) return fail();
    int k = 0;
    for (int64_t n : sizes) {
      if (n >= 0 && t.size(k) != n) return fail();
      ++k;
    }
    if (device < 0) device = t.get_device();
    return &t;
  }
  template <class T = void>
  T* data(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> sizes) {
    if (o == Py_None) return nullptr;
    const at::Tensor* t = tensor(o, type, sizes);
    return t ? static_cast<T*>(t->data_ptr()) : nullptr;
  }
  // a workspace: bytes of any number
  void* bytes(PyObject* o, size_t& n) {
    n = 0;
    if (o == Py_None) return nullptr;
    const at::Tensor* t = tensor(o, at::kByte, {-1});
    if (!t) return nullptr;
    n = (size_t)t->numel();
    return t->data_ptr();
  }
  float number(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) fail();
    return (float)v;
  }
  void* stream() {
    if (!ok || device < 0) { fail(); return nullptr; }
    PyObject* index = PyLong_FromLong(device);
    PyObject* r = index ? PyObject_CallFunctionObjArgs(g_stream_of, index, nullptr) : nullptr;
    Py_XDECREF(index);
    if (!r) { fail(); return nullptr; }
    void* st = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) fail();
    return st;
  }
  const at::Tensor* fail() { ok = false; return nullptr; }
};

// The C structure behind a ctypes one of the given type (other objects may have as many bytes).
template <class S>
struct Struct {
  Py_buffer view{};
  bool ok;
  Struct(PyObject* o, PyObject* type)
      : ok(type && PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(type)) && PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0) {
    if (ok && view.len != (Py_ssize_t)sizeof(S)) { PyBuffer_Release(&view); ok = false; }
  }
  ~Struct() { if (ok) PyBuffer_Release(&view); }
  const S* get() const { return static_cast<const S*>(view.buf); }
};

PyObject* not_here() {
  PyErr_Clear();
  Py_RETURN_NONE;
}
// (torch reports some tensors without memory of their own by an exception)
template <class F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (...) {
    return not_here();
  }
}
struct WithoutGil {   // (given back also where the call ends by an exception)
  PyThreadState* state = PyEval_SaveThread();
  ~WithoutGil() { PyEval_RestoreThread(state); }
};
// An exception out of the library is the call's result: it may have enqueued work, so the call is not made again.
template <class F>
PyObject* finish(Call& c, F&& call) {
  if (!c.ok) return not_here();
  int rc;
  try {
    WithoutGil released;
    rc = call();
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  } catch (...) {
    PyErr_SetString(PyExc_RuntimeError, "exception in the library");
    return nullptr;
  }
  return PyLong_FromLong(rc);
}

constexpr auto kBf16 = at::kBFloat16;
constexpr auto kI32 = at::kInt;
at::ScalarType out_type(int32_t out_dtype) { return out_dtype == MARL_OUT_BF16 ? kBf16 : at::kFloat; }

// shape, workspace, q, k_pages, v_pages, prefix_block_table, suffix_block_table, prefix_lens, suffix_lens, group_of_seq, scale, out
PyObject* decode_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 12 || !f_decode_attn) Py_RETURN_NONE;
    Struct<marl_attn_shape> s(a[0], g_attn_shape);
    if (!s.ok) return not_here();
    const marl_attn_shape& h = *s.get();
    if (a[1] == Py_None || a[11] == Py_None) return not_here();
    if (h.max_prefix_pages <= 0 || h.max_suffix_pages <= 0) return not_here();   // (tables whose extents are not looked at)
    Call c;
    void* out = c.data(a[11], out_type(h.out_dtype), {h.num_seqs, h.num_q_heads, 128});   // (first: the call's device)
    size_t bytes;
    void* ws = c.bytes(a[1], bytes);
    const void* q = c.data(a[2], kBf16, {h.num_seqs, h.num_q_heads, 128});
    const void* k = c.data(a[3], kBf16, {h.num_pages, h.num_kv_heads, 16, 128});
    const void* v = c.data(a[4], kBf16, {h.num_pages, h.num_kv_heads, 128, 16});
    const int32_t* pt = c.data<int32_t>(a[5], kI32, {h.num_groups, h.max_prefix_pages});
    const int32_t* st = c.data<int32_t>(a[6], kI32, {h.num_seqs, h.max_suffix_pages});
    const int32_t* pl = c.data<int32_t>(a[7], kI32, {h.num_groups});
    const int32_t* sl = c.data<int32_t>(a[8], kI32, {h.num_seqs});
    const int32_t* gs = c.data<int32_t>(a[9], kI32, {h.num_seqs});
    const float scale = c.number(a[10]);
    void* stream = c.stream();
    return finish(c, [&] { return f_decode_attn(&h, ws, bytes, q, k, v, pt, st, pl, sl, gs, scale, out, stream); });
  });
}

// logits, tokens, temperature, out, workspace
PyObject* token_logprobs(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 5 || !f_token_logprobs) Py_RETURN_NONE;
    Call c;
    const at::Tensor* x = c.tensor(a[0], kBf16, {-1, -1});
    if (!x || a[1] == Py_None || a[3] == Py_None) return not_here();
    const int64_t rows = x->size(0), vocab = x->size(1);
    if (rows > INT32_MAX || vocab > INT32_MAX) return not_here();
    const int32_t* tokens = c.data<int32_t>(a[1], kI32, {rows});
    const float temperature = c.number(a[2]);
    float* out = c.data<float>(a[3], at::kFloat, {rows});
    size_t bytes;
    void* ws = c.bytes(a[4], bytes);
    void* stream = c.stream();
    return finish(c, [&] { return f_token_logprobs(x->data_ptr(), tokens, temperature, out, (int32_t)rows, (int32_t)vocab, ws, bytes, stream); });
  });
}

// logits, uniforms, temperature, top_p or None, out_tokens, out_logprobs, workspace (not with top_p)
PyObject* sample_tokens(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 7 || !f_sample_tokens || !f_sample_tokens_top_p) Py_RETURN_NONE;
    Call c;
    const at::Tensor* x = c.tensor(a[0], kBf16, {-1, -1});
    const bool nucleus = a[3] != Py_None;
    if (!x || a[1] == Py_None || a[4] == Py_None || a[5] == Py_None || (!nucleus && a[6] == Py_None)) return not_here();
    const int64_t rows = x->size(0), vocab = x->size(1);
    if (rows > INT32_MAX || vocab > INT32_MAX) return not_here();
    const float* u = c.data<float>(a[1], at::kFloat, {rows});
    const float temperature = c.number(a[2]);
    int32_t* tokens = c.data<int32_t>(a[4], kI32, {rows});
    float* logprobs = c.data<float>(a[5], at::kFloat, {rows});
    const void* logits = x->data_ptr();
    if (nucleus) {
      const float top_p = c.number(a[3]);
      void* stream = c.stream();
      return finish(c, [&] { return f_sample_tokens_top_p(logits, u, temperature, top_p, tokens, logprobs, (int32_t)rows, (int32_t)vocab, stream); });
    }
    size_t bytes;
    void* ws = c.bytes(a[6], bytes);
    void* stream = c.stream();
    return finish(c, [&] { return f_sample_tokens(logits, u, temperature, tokens, logprobs, (int32_t)rows, (int32_t)vocab, ws, bytes, stream); });
  });
}

// shape, k_new, v_new, k_pages, v_pages, suffix_block_table, suffix_lens, flags
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 8 || !f_kv_append) Py_RETURN_NONE;
    Struct<marl_attn_shape> s(a[0], g_attn_shape);
    if (!s.ok || a[3] == Py_None || a[7] != Py_None) return not_here();
    const marl_attn_shape& h = *s.get();
    Call c;
    void* k = c.data(a[3], kBf16, {h.num_pages, h.num_kv_heads, 16, 128});
    void* v = c.data(a[4], kBf16, {h.num_pages, h.num_kv_heads, 128, 16});
    const void* kn = c.data(a[1], kBf16, {h.num_seqs, h.num_kv_heads, 128});
    const void* vn = c.data(a[2], kBf16, {h.num_seqs, h.num_kv_heads, 128});
    const int32_t* st = c.data<int32_t>(a[5], kI32, {h.num_seqs, h.max_suffix_pages});
    int32_t* sl = c.data<int32_t>(a[6], kI32, {h.num_seqs});
    void* stream = c.stream();
    return finish(c, [&] { return f_kv_append(&h, kn, vn, k, v, st, sl, nullptr, stream); });
  });
}

// shape, workspace, q, k_pages, v_pages, prefix_block_table, q_start, q_pos0, scale, out
PyObject* prefill_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 10 || !f_prefill_attn) Py_RETURN_NONE;
    Struct<marl_prefill_shape> s(a[0], g_prefill_shape);
    if (!s.ok || a[1] == Py_None || a[2] == Py_None) return not_here();
    const marl_prefill_shape& h = *s.get();
    Call c;
    const void* q = c.data(a[2], kBf16, {h.num_tokens, h.num_q_heads, 128});   // (first: the call's device)
    size_t bytes;
    void* ws = c.bytes(a[1], bytes);
    const void* k = c.data(a[3], kBf16, {h.num_pages, h.num_kv_heads, 16, 128});
    const void* v = c.data(a[4], kBf16, {h.num_pages, h.num_kv_heads, 128, 16});
    const int32_t* pt = c.data<int32_t>(a[5], kI32, {h.num_groups, h.max_prefix_pages});
    const int32_t* qs = c.data<int32_t>(a[6], kI32, {(int64_t)h.num_groups + 1});
    const int32_t* qp = c.data<int32_t>(a[7], kI32, {h.num_groups});
    const float scale = c.number(a[8]);
    void* out = c.data(a[9], out_type(h.out_dtype), {h.num_tokens, h.num_q_heads, 128});
    void* stream = c.stream();
    return finish(c, [&] { return f_prefill_attn(&h, ws, bytes, q, k, v, pt, qs, qp, scale, out, stream); });
  });
}

// shape, k_new, v_new, k_pages, v_pages, prefix_block_table, q_start, q_pos0, flags
PyObject* kv_write_prompt(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 9 || !f_kv_write_prompt) Py_RETURN_NONE;
    Struct<marl_prefill_shape> s(a[0], g_prefill_shape);
    if (!s.ok || a[1] == Py_None || a[8] != Py_None) return not_here();
    const marl_prefill_shape& h = *s.get();
    Call c;
    const void* kn = c.data(a[1], kBf16, {h.num_tokens, h.num_kv_heads, 128});   // (first: the call's device)
    const void* vn = c.data(a[2], kBf16, {h.num_tokens, h.num_kv_heads, 128});
    void* k = c.data(a[3], kBf16, {h.num_pages, h.num_kv_heads, 16, 128});
    void* v = c.data(a[4], kBf16, {h.num_pages, h.num_kv_heads, 128, 16});
    const int32_t* pt = c.data<int32_t>(a[5], kI32, {h.num_groups, h.max_prefix_pages});
    const int32_t* qs = c.data<int32_t>(a[6], kI32, {(int64_t)h.num_groups + 1});
    const int32_t* qp = c.data<int32_t>(a[7], kI32, {h.num_groups});
    void* stream = c.stream();
    return finish(c, [&] { return f_kv_write_prompt(&h, kn, vn, k, v, pt, qs, qp, nullptr, stream); });
  });
}

// bind(stream_of, types of the two shapes, addresses of the library's functions in the order of the declarations above; the
// scatter's may be left out and then stays what it is)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n < 9 || n > 10 || !PyType_Check(a[1]) || !PyType_Check(a[2])) {
    PyErr_SetString(PyExc_TypeError, "bind: a function, two types, six or seven addresses");
    return nullptr;
  }
  void* f[7] = {};
  for (int k = 0; k + 3 < n; ++k) {
    f[k] = PyLong_AsVoidPtr(a[k + 3]);
    if (PyErr_Occurred()) return nullptr;
  }
  PyObject** const kept[3] = {&g_stream_of, &g_attn_shape, &g_prefill_shape};
  for (int k = 0; k < 3; ++k) {
    Py_INCREF(a[k]);
    Py_XSETREF(*kept[k], a[k]);
  }
  f_decode_attn = reinterpret_cast<decltype(f_decode_attn)>(f[0]);
  f_token_logprobs = reinterpret_cast<decltype(f_token_logprobs)>(f[1]);
  f_kv_append = reinterpret_cast<decltype(f_kv_append)>(f[2]);
  f_sample_tokens = reinterpret_cast<decltype(f_sample_tokens)>(f[3]);
  f_sample_tokens_top_p = reinterpret_cast<decltype(f_sample_tokens_top_p)>(f[4]);
  f_prefill_attn = reinterpret_cast<decltype(f_prefill_attn)>(f[5]);
  if (n == 10) f_kv_write_prompt = reinterpret_cast<decltype(f_kv_write_prompt)>(f[6]);
  Py_RETURN_NONE;
}

#define MARL_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MARL_FAST(bind), MARL_FAST(decode_attn), MARL_FAST(token_logprobs), MARL_FAST(sample_tokens),
                         MARL_FAST(kv_append), MARL_FAST(prefill_attn), MARL_FAST(kv_write_prompt), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "fast_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_fast_calls(void) {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) != 0) Py_CLEAR(m);   // (tensors are read as this torch lays them out)
  if (m && PyModule_AddStringConstant(m, "sources", MARL_FAST_CALLS_SOURCES) != 0) Py_CLEAR(m);
  return m;
}
