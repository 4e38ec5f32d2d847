// The hot calls of paper_2603_05353_amd.Layer from Python objects to the C ABI without an interpreter step per argument: a
// small layer's launches take the GPU less time than the checks of its tensors took the interpreter (a 1024-key layer of
// 4 chunks 41 us of host work for 38 us of kernels, of which 20 us were marshalling; 16 chunks 61 us, 41).
//
// Only what is plainly right is taken here: exact tensors on the GPU of the expected type, shape and layout, whole numbers that
// fit.  Anything else -- also every mistake -- returns None before any C call is made, and the caller goes the way through the
// interpreter, which knows the message.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cstdint>
#include <exception>
#include <limits>
#include <string>
#include <vector>

#include "ifkv.h"

namespace {

struct Caller {
  PyObject_HEAD
  ifkv_ctx *ctx;
  at::ScalarType dtype;
  int64_t n_q_heads, n_kv_heads, head_dim, token_stride, head_stride;
  decltype(&ifkv_reposition_keys) reposition_keys;
  decltype(&ifkv_reposition_score) reposition_score;
  decltype(&ifkv_score_tokens) score_tokens;
  decltype(&ifkv_select_topk) select_topk;
  decltype(&ifkv_recompute_attention) recompute_attention;
  decltype(&ifkv_splice_kv) splice_kv;
  decltype(&ifkv_rope_rows) rope_rows;
};

// A tensor's address if it is what the C call expects; `ok` is cleared otherwise.
struct Args {
  bool ok = true;
  void *packed(PyObject *o, at::ScalarType dtype, std::initializer_list<int64_t> tail, int64_t rows) {
    const at::Tensor *t = plain(o, dtype);
    if (t == nullptr || t->dim() != static_cast<int64_t>(tail.size()) + 1 || t->size(0) < rows || !t->is_contiguous()) return refuse();
    int64_t i = 1;
    for (int64_t n : tail)
      if (t->size(i++) != n) return refuse();
    return t->data_ptr();
  }
  void *cache(PyObject *o, const Caller *c, int64_t rows = 0) {
    const at::Tensor *t = plain(o, c->dtype);
    if (t == nullptr || t->dim() != 3 || t->size(0) < rows || t->size(1) != c->n_kv_heads || t->size(2) != c->head_dim) return refuse();
    if (t->size(0) > 1 && (t->stride(0) != c->token_stride || t->stride(1) != c->head_stride || t->stride(2) != 1)) return refuse();
    return t->data_ptr();
  }
  // rows of any tensor
  int64_t rows(PyObject *o) {
    if (!THPVariable_CheckExact(o) || THPVariable_Unpack(o).dim() < 1) {
      ok = false;
      return 0;
    }
    return THPVariable_Unpack(o).size(0);
  }
  int64_t number(PyObject *o, int64_t lo, int64_t hi) {
    if (!PyLong_CheckExact(o) && !PyBool_Check(o)) {
      ok = false;
      return 0;
    }
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow != 0 || v < lo || v > hi) {
      ok = false;
      return 0;
    }
    return v;
  }
  template <typename T>
  const T *numbers(PyObject *o, Py_ssize_t n, std::vector<T> &out) {
    if (o == Py_None) return nullptr;
    if ((!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) || PySequence_Fast_GET_SIZE(o) != n) {
      ok = false;
      return nullptr;
    }
    out.resize(n + 1);
    for (Py_ssize_t i = 0; i < n; ++i)
      out[i] = static_cast<T>(number(PySequence_Fast_GET_ITEM(o, i), std::numeric_limits<T>::min(), std::numeric_limits<T>::max()));
    return out.data();
  }

 private:
  void *refuse() {
    ok = false;
    return nullptr;
  }
  const at::Tensor *plain(PyObject *o, at::ScalarType dtype) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.has_storage() && t.layout() == at::kStrided && t.is_cuda() && t.scalar_type() == dtype ? &t : nullptr;
  }
};

PyObject *none() { Py_RETURN_NONE; }

// The C call threw: the Python error is set.
struct CallFailed {};

// Runs f, which checks and calls; None where it refuses or a tensor throws.  Neither here nor in without_gil is anything caught that is
// not an exception: a thread that comes back when the interpreter is on its way out is ended by unwinding its stack.
template <typename F>
PyObject *guarded(F f) {
  try {
    return f();
  } catch (const CallFailed &) {
    return nullptr;
  } catch (const std::exception &) {
    PyErr_Clear();
    return none();
  }
}

// f touches no Python object
template <typename F>
int without_gil(F f) {
  PyThreadState *state = PyEval_SaveThread();
  int rc = 0;
  std::string failure;
  bool failed = false;
  try {
    rc = f();
  } catch (const std::exception &e) {
    failed = true;
    failure = e.what();
  }
  PyEval_RestoreThread(state);  // (not in a destructor, for the same reason)
  if (failed) {
    PyErr_SetString(PyExc_RuntimeError, failure.c_str());
    throw CallFailed{};
  }
  return rc;
}

constexpr int64_t kInt32 = std::numeric_limits<int32_t>::max();

// (k_chunks, v_chunks, chunk_order, cached_pos0, delta_override, k_out, v_out [, q_prompt, k_prompt, scores, accumulate])
// -> None or (rc, starts, n_ctx)
PyObject *reposition(Caller *self, PyObject *const *a, bool score) {
  return guarded([&]() -> PyObject * {
    PyObject *kl = a[0], *vl = a[1];
    if (!PyList_CheckExact(kl) && !PyTuple_CheckExact(kl)) return none();
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(kl);
    const bool has_v = vl != Py_None;
    if (n > kInt32 || (has_v && ((!PyList_CheckExact(vl) && !PyTuple_CheckExact(vl)) || PySequence_Fast_GET_SIZE(vl) != n))) return none();
    Args x;
    std::vector<const void *> k(n + 1), v(n + 1);
    std::vector<int32_t> len(n + 1), order, pos0;
    std::vector<int64_t> delta, start(n + 1);
    int64_t total = 0;
    for (Py_ssize_t i = 0; i < n && x.ok; ++i) {
      PyObject *ko = PySequence_Fast_GET_ITEM(kl, i);
      const int64_t rows = x.rows(ko);
      if (rows > kInt32) return none();
      len[i] = static_cast<int32_t>(rows);
      total += rows;
      if (rows > 0) k[i] = x.packed(ko, self->dtype, {self->n_kv_heads, self->head_dim}, 0);
      if (has_v) {
        PyObject *vo = PySequence_Fast_GET_ITEM(vl, i);
        if (x.rows(vo) != rows) return none();
        if (rows > 0) v[i] = x.packed(vo, self->dtype, {self->n_kv_heads, self->head_dim}, 0);
      }
    }
    if (!x.ok) return none();
    const int32_t *order_p = x.numbers(a[2], n, order), *pos0_p = x.numbers(a[3], n, pos0);
    const int64_t *delta_p = x.numbers(a[4], n, delta);
    void *k_out = x.cache(a[5], self), *v_out = a[6] == Py_None ? nullptr : x.cache(a[6], self);
    if (!x.ok || x.rows(a[5]) < total || (a[6] != Py_None && x.rows(a[6]) < total)) return none();
    int64_t n_ctx = 0;
    int rc;
    if (score) {
      const int64_t m = x.rows(a[7]);
      const void *q = x.packed(a[7], self->dtype, {self->n_q_heads, self->head_dim}, 0);
      const void *kp = a[8] == Py_None ? nullptr : x.packed(a[8], self->dtype, {self->n_kv_heads, self->head_dim}, m);
      float *scores = static_cast<float *>(x.packed(a[9], at::kFloat, {}, total));
      const int64_t accumulate = x.number(a[10], 0, 1);
      if (!x.ok || m > kInt32) return none();
      rc = without_gil([&] {
        return self->reposition_score(self->ctx, static_cast<int32_t>(n), k.data(), has_v ? v.data() : nullptr, len.data(), order_p, pos0_p,
                                      delta_p, k_out, v_out, start.data(), &n_ctx, q, static_cast<int32_t>(m), kp,
                                      static_cast<int32_t>(accumulate), scores);
      });
    } else {
      rc = without_gil([&] {
        return self->reposition_keys(self->ctx, static_cast<int32_t>(n), k.data(), has_v ? v.data() : nullptr, len.data(), order_p, pos0_p,
                                     delta_p, k_out, v_out, start.data(), &n_ctx);
      });
    }
    PyObject *starts = PyList_New(n);
    if (starts == nullptr) return nullptr;
    for (Py_ssize_t i = 0; i < n; ++i) {
      PyObject *s = PyLong_FromLongLong(start[i]);
      if (s == nullptr) {
        Py_DECREF(starts);
        return nullptr;
      }
      PyList_SET_ITEM(starts, i, s);
    }
    return Py_BuildValue("(iNL)", rc, starts, static_cast<long long>(n_ctx));
  });
}

PyObject *wrong_count() {
  PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
  return nullptr;
}

PyObject *call_reposition_keys(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  return n == 7 ? reposition(reinterpret_cast<Caller *>(self), a, false) : wrong_count();
}
PyObject *call_reposition_score(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  return n == 11 ? reposition(reinterpret_cast<Caller *>(self), a, true) : wrong_count();
}

// (k_global, q_prompt, k_prompt, scores, accumulate)
PyObject *call_score_tokens(PyObject *o, PyObject *const *a, Py_ssize_t n) {
  Caller *self = reinterpret_cast<Caller *>(o);
  if (n != 5) return wrong_count();
  return guarded([&]() -> PyObject * {
    Args x;
    const void *k = x.cache(a[0], self), *q = x.packed(a[1], self->dtype, {self->n_q_heads, self->head_dim}, 0);
    if (!x.ok) return none();
    const int64_t n_ctx = x.rows(a[0]), m = x.rows(a[1]);
    const void *kp = a[2] == Py_None ? nullptr : x.packed(a[2], self->dtype, {self->n_kv_heads, self->head_dim}, m);
    float *scores = static_cast<float *>(x.packed(a[3], at::kFloat, {}, n_ctx));
    const int64_t accumulate = x.number(a[4], 0, 1);
    if (!x.ok || m > kInt32) return none();
    return PyLong_FromLong(without_gil([&] {
      return self->score_tokens(self->ctx, k, n_ctx, q, static_cast<int32_t>(m), kp, static_cast<int32_t>(accumulate), scores);
    }));
  });
}

// (scores, ratio, k, idx_out) -> None or (rc, k)
PyObject *call_select_topk(PyObject *o, PyObject *const *a, Py_ssize_t n) {
  Caller *self = reinterpret_cast<Caller *>(o);
  if (n != 4) return wrong_count();
  return guarded([&]() -> PyObject * {
    Args x;
    const float *scores = static_cast<const float *>(x.packed(a[0], at::kFloat, {}, 0));
    int32_t *idx = static_cast<int32_t *>(x.packed(a[3], at::kInt, {}, 0));
    const int64_t k = x.number(a[2], std::numeric_limits<int64_t>::min(), std::numeric_limits<int64_t>::max());
    if (!x.ok || !PyFloat_CheckExact(a[1])) return none();
    int64_t k_out = 0;
    const int64_t n_ctx = x.rows(a[0]), n_idx = x.rows(a[3]);
    const double ratio = PyFloat_AS_DOUBLE(a[1]);
    // without a buffer the call reports k and does nothing else: the buffer has to hold that many
    int rc = self->select_topk(self->ctx, scores, n_ctx, ratio, k, nullptr, &k_out);
    if (rc == IFKV_OK) {
      if (n_idx < k_out) return none();
      rc = without_gil([&] { return self->select_topk(self->ctx, scores, n_ctx, ratio, k, idx, &k_out); });
    }
    return Py_BuildValue("(iL)", rc, static_cast<long long>(k_out));
  });
}

// (q_sel, row_pos, k_cache, v_cache, out, lse)
PyObject *call_recompute_attention(PyObject *o, PyObject *const *a, Py_ssize_t n) {
  Caller *self = reinterpret_cast<Caller *>(o);
  if (n != 6) return wrong_count();
  return guarded([&]() -> PyObject * {
    Args x;
    const void *q = x.packed(a[0], self->dtype, {self->n_q_heads, self->head_dim}, 0);
    const int64_t rows = x.rows(a[0]), n_kv = x.rows(a[2]);
    const void *k = x.cache(a[2], self), *v = x.cache(a[3], self, n_kv);
    if (!x.ok) return none();
    const int32_t *pos = static_cast<const int32_t *>(x.packed(a[1], at::kInt, {}, rows));
    void *out = x.packed(a[4], self->dtype, {self->n_q_heads, self->head_dim}, rows);
    float *lse = a[5] == Py_None ? nullptr : static_cast<float *>(x.packed(a[5], at::kFloat, {self->n_q_heads}, rows));
    if (!x.ok) return none();
    return PyLong_FromLong(without_gil([&] { return self->recompute_attention(self->ctx, q, pos, rows, k, v, n_kv, out, lse); }));
  });
}

// (k_new, v_new, idx, k_cache, v_cache)
PyObject *call_splice_kv(PyObject *o, PyObject *const *a, Py_ssize_t n) {
  Caller *self = reinterpret_cast<Caller *>(o);
  if (n != 5) return wrong_count();
  return guarded([&]() -> PyObject * {
    Args x;
    const int32_t *idx = static_cast<const int32_t *>(x.packed(a[2], at::kInt, {}, 0));
    const int64_t rows = x.rows(a[2]), n_kv = x.rows(a[3]);
    void *k = x.cache(a[3], self), *v = a[4] == Py_None ? nullptr : x.cache(a[4], self, n_kv);
    if (!x.ok) return none();
    const void *kn = x.packed(a[0], self->dtype, {self->n_kv_heads, self->head_dim}, rows);
    const void *vn = a[1] == Py_None ? nullptr : x.packed(a[1], self->dtype, {self->n_kv_heads, self->head_dim}, rows);
    if (!x.ok) return none();
    return PyLong_FromLong(without_gil([&] { return self->splice_kv(self->ctx, kn, vn, idx, rows, k, v, n_kv); }));
  });
}

// (x, pos)
PyObject *call_rope_rows(PyObject *o, PyObject *const *a, Py_ssize_t n) {
  Caller *self = reinterpret_cast<Caller *>(o);
  if (n != 2) return wrong_count();
  return guarded([&]() -> PyObject * {
    Args x;
    if (!THPVariable_CheckExact(a[0]) || THPVariable_Unpack(a[0]).dim() != 3) return none();
    const int64_t rows = x.rows(a[0]), heads = THPVariable_Unpack(a[0]).size(1);
    void *t = x.packed(a[0], self->dtype, {heads, self->head_dim}, 0);
    const int32_t *pos = static_cast<const int32_t *>(x.packed(a[1], at::kInt, {}, rows));
    if (!x.ok || heads > kInt32) return none();
    return PyLong_FromLong(without_gil([&] { return self->rope_rows(self->ctx, t, pos, rows, static_cast<int32_t>(heads)); }));
  });
}

// Caller(ctx, bf16, n_q_heads, n_kv_heads, head_dim, token_stride, head_stride, seven addresses in the order of the struct)
PyObject *caller_new(PyTypeObject *type, PyObject *args, PyObject *) {
  unsigned long long p[8];
  int bf16;
  long long d[5];
  if (!PyArg_ParseTuple(args, "KpLLLLLKKKKKKK", &p[0], &bf16, &d[0], &d[1], &d[2], &d[3], &d[4], &p[1], &p[2], &p[3], &p[4], &p[5], &p[6], &p[7]))
    return nullptr;
  PyObject *o = type->tp_alloc(type, 0);
  if (o == nullptr) return nullptr;
  Caller *c = reinterpret_cast<Caller *>(o);
  c->ctx = reinterpret_cast<ifkv_ctx *>(p[0]);
  c->dtype = bf16 ? at::kBFloat16 : at::kFloat;
  c->n_q_heads = d[0];
  c->n_kv_heads = d[1];
  c->head_dim = d[2];
  c->token_stride = d[3];
  c->head_stride = d[4];
  c->reposition_keys = reinterpret_cast<decltype(c->reposition_keys)>(p[1]);
  c->reposition_score = reinterpret_cast<decltype(c->reposition_score)>(p[2]);
  c->score_tokens = reinterpret_cast<decltype(c->score_tokens)>(p[3]);
  c->select_topk = reinterpret_cast<decltype(c->select_topk)>(p[4]);
  c->recompute_attention = reinterpret_cast<decltype(c->recompute_attention)>(p[5]);
  c->splice_kv = reinterpret_cast<decltype(c->splice_kv)>(p[6]);
  c->rope_rows = reinterpret_cast<decltype(c->rope_rows)>(p[7]);
  return o;
}

#define IFKV_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(call_##name)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {IFKV_METHOD(reposition_keys), IFKV_METHOD(reposition_score), IFKV_METHOD(score_tokens), IFKV_METHOD(select_topk),
                          IFKV_METHOD(recompute_attention), IFKV_METHOD(splice_kv), IFKV_METHOD(rope_rows), {nullptr, nullptr, 0, nullptr}};
#undef IFKV_METHOD

PyTypeObject kCallerType = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_ifkv_marshal", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ifkv_marshal() {
  kCallerType.tp_name = "_ifkv_marshal.Caller";
  kCallerType.tp_basicsize = sizeof(Caller);
  kCallerType.tp_flags = Py_TPFLAGS_DEFAULT;
  kCallerType.tp_methods = kMethods;
  kCallerType.tp_new = caller_new;
  if (PyType_Ready(&kCallerType) < 0) return nullptr;
  PyObject *m = PyModule_Create(&kModule);
  if (m == nullptr) return nullptr;
  // the layout of objects and tensors is that of the headers this was compiled with
  if (PyModule_AddIntConstant(m, "python_version", PY_VERSION_HEX >> 16) < 0 || PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  Py_INCREF(&kCallerType);
  if (PyModule_AddObject(m, "Caller", reinterpret_cast<PyObject *>(&kCallerType)) < 0) {
    Py_DECREF(&kCallerType);
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
