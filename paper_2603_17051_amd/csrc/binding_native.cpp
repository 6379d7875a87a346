// The Python binding's calls that run once per layer and step, as a CPython module: the tensors of a call are checked and
// their addresses taken here, then the C ABI is called.  A small call is bound by its host work, of which checks,
// attribute reads and ctypes conversions in Python were about half: us of host time, Python / here, forward 7.6 / 4.3, forward
// and backward 15.5 / 8.3, loss 11.5 / 6.6, a cache of three appends rebuilt 18.6 / 13.3.
//
// Every function answers None, with nothing done, for a call it does not take as it is: an argument left out, a
// tensor that is not plain or does not match, a number of another type.  binding.py then goes through its own
// checks, which raise what there is to raise.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "../../include/astro.h"

namespace {

struct Library {  // the functions of the library that binding.py has loaded
  decltype(&astro_kvcache_append) append;
  decltype(&astro_chunk_attn_fwd) chunk_fwd;
  decltype(&astro_group_attn_fwd) group_fwd;
  decltype(&astro_chunk_attn_bwd) chunk_bwd;
  decltype(&astro_group_attn_bwd) group_bwd;
  decltype(&astro_chunk_attn_bwd_full) bwd_full;
  decltype(&astro_nft_loss_workspace_bytes) loss_workspace_bytes;
  decltype(&astro_nft_loss) loss;
} lib;

// What a call's arguments are read through: `ok` turns false at the first that this module does not take.
struct Reader {
  bool ok = true;
  int64_t batch = 0, tokens = 0, heads = 0, head_dim = 0;  // of the cache
  at::ScalarType dtype = at::kBFloat16;

  // an astro_kvcache_t* held in a ctypes.c_void_p
  astro_kvcache_t* handle(PyObject* o) {
    static PyObject* const name = PyUnicode_InternFromString("value");
    PyObject* v = PyObject_GetAttr(o, name);
    void* p = v && PyLong_CheckExact(v) ? PyLong_AsVoidPtr(v) : nullptr;
    Py_XDECREF(v);
    if (PyErr_Occurred()) PyErr_Clear();
    ok = ok && p;
    return static_cast<astro_kvcache_t*>(p);
  }
  int64_t integer(PyObject* o, int64_t most) {
    int overflow = 0;
    const int64_t v = PyLong_CheckExact(o) ? PyLong_AsLongLongAndOverflow(o, &overflow) : -1;
    ok = ok && !overflow && v >= 0 && v <= most;
    return v;
  }
  float number(PyObject* o) {
    ok = ok && PyFloat_CheckExact(o);
    return ok ? (float)PyFloat_AS_DOUBLE(o) : 0.f;
  }
  // (batch, tokens of a frame, heads, head dim, whether bf16)
  void dims(PyObject* o) {
    ok = ok && PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 5;
    if (!ok) return;
    int64_t* to[4] = {&batch, &tokens, &heads, &head_dim};
    for (int i = 0; i < 4; ++i) *to[i] = integer(PyTuple_GET_ITEM(o, i), INT32_MAX);
    dtype = PyTuple_GET_ITEM(o, 4) == Py_True ? at::kBFloat16 : at::kFloat;
  }
  // a plain tensor in device memory
  const at::Tensor* plain(PyObject* o) {
    ok = ok && THPVariable_CheckExact(o) && THPVariable_Unpack(o).is_cuda();
    return ok ? &THPVariable_Unpack(o) : nullptr;
  }
  void* of_type(PyObject* o, at::ScalarType type, int64_t numel) {
    const at::Tensor* t = plain(o);
    ok = ok && t->scalar_type() == type && t->numel() == numel && t->is_contiguous();
    return ok ? t->data_ptr() : nullptr;
  }
  // the log-sum-exps of `rows` queries; a call without candidates also takes a longer buffer
  float* lse(PyObject* o, int64_t rows, bool longer) {
    const at::Tensor* t = plain(o);
    ok = ok && t->scalar_type() == at::kFloat && t->is_contiguous() && (t->numel() == rows || (longer && t->numel() > rows));
    return ok ? static_cast<float*>(t->data_ptr()) : nullptr;
  }
  // a contiguous tensor [rows, tokens, heads, head dim]
  void* rows(PyObject* o, at::ScalarType type, int64_t n_batch, int64_t n_rows) {
    const at::Tensor* t = plain(o);
    if (!t) return nullptr;
    const at::IntArrayRef s = t->sizes();
    ok = t->scalar_type() == type && s.size() == 4 && s[0] == n_batch && s[1] == n_rows && s[2] == heads &&
         s[3] == head_dim && t->is_contiguous();
    return ok ? t->data_ptr() : nullptr;
  }
  void* workspace(PyObject* o, size_t* bytes) {
    const at::Tensor* t = plain(o);
    if (!t) return nullptr;
    *bytes = (size_t)t->numel() * t->element_size();
    return t->data_ptr();
  }
};

struct WithoutLock {  // the interpreter's, also given back when something throws
  PyThreadState* const state = PyEval_SaveThread();
  ~WithoutLock() { PyEval_RestoreThread(state); }
};

// runs `call` on the current stream
template <typename F>
PyObject* run(F call) {
  void* const stream = (void*)c10::hip::getCurrentHIPStream().stream();
  int code;
  {
    WithoutLock w;
    code = call(stream);
  }
  return PyLong_FromLong(code);
}

// what a tensor without storage and its like throw: the call is left to Python
template <typename F>
PyObject* guarded(F body) {
  try {
    if (PyObject* r = body()) return r;
  } catch (...) {
  }
  Py_RETURN_NONE;
}

// (handle, dims, k, v, n_frames)
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 5) return nullptr;
    Reader r;
    astro_kvcache_t* const cache = r.handle(a[0]);
    r.dims(a[1]);
    const int64_t frames = r.integer(a[4], INT32_MAX);
    void* const k = r.rows(a[2], r.dtype, r.batch, frames * r.tokens);
    void* const v = r.rows(a[3], r.dtype, r.batch, frames * r.tokens);
    if (!r.ok) return nullptr;
    return run([&](void* s) { return lib.append(cache, k, v, (int32_t)frames, s); });
  });
}

// (handle, dims, q, k_chunk, v_chunk, n_frames, group, out, lse, workspace); group 0: the call without candidates
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 10) return nullptr;
    Reader r;
    astro_kvcache_t* const cache = r.handle(a[0]);
    r.dims(a[1]);
    const int64_t frames = r.integer(a[5], INT32_MAX), group = r.integer(a[6], INT32_MAX);
    const int64_t batch = r.batch * (group ? group : 1), rows = frames * r.tokens;
    void* t[4];
    PyObject* const from[4] = {a[2], a[3], a[4], a[7]};
    for (int i = 0; i < 4; ++i) t[i] = r.rows(from[i], r.dtype, batch, rows);
    float* const lse = r.lse(a[8], batch * r.heads * rows, !group);
    size_t bytes = 0;
    void* const ws = r.workspace(a[9], &bytes);
    if (!r.ok) return nullptr;
    return run([&](void* s) {
      return group ? lib.group_fwd(cache, t[0], t[1], t[2], (int32_t)frames, (int32_t)group, t[3], lse, ws, bytes, s)
                   : lib.chunk_fwd(cache, t[0], t[1], t[2], (int32_t)frames, t[3], lse, ws, bytes, s);
    });
  });
}

// (handle, dims, q, k_chunk, v_chunk, out, lse, dout, n_frames, group, dq, dk_chunk, dv_chunk, workspace) as above, or
// with (..., dk_cache, dv_cache, capacity_frames) behind, group 0: the non-detached backward
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 14 && n != 17) return nullptr;
    Reader r;
    astro_kvcache_t* const cache = r.handle(a[0]);
    r.dims(a[1]);
    const int64_t frames = r.integer(a[8], INT32_MAX), group = r.integer(a[9], INT32_MAX);
    const int64_t batch = r.batch * (group ? group : 1), rows = frames * r.tokens;
    void *t[5], *grad[5] = {};
    PyObject* const from[5] = {a[2], a[3], a[4], a[5], a[7]};
    for (int i = 0; i < 5; ++i) t[i] = r.rows(from[i], r.dtype, batch, rows);
    for (int i = 0; i < 3; ++i) grad[i] = r.rows(a[10 + i], at::kFloat, batch, rows);
    if (n == 17) {
      const int64_t capacity = r.integer(a[16], INT32_MAX);
      for (int i = 0; i < 2; ++i) grad[3 + i] = r.rows(a[14 + i], at::kFloat, r.batch, capacity * r.tokens);
    }
    float* const lse = r.lse(a[6], batch * r.heads * rows, !group);
    size_t bytes = 0;
    void* const ws = r.workspace(a[13], &bytes);
    if (!r.ok) return nullptr;
    float** const g = (float**)grad;
    return run([&](void* s) {
      if (n == 17)
        return lib.bwd_full(cache, t[0], t[1], t[2], t[3], lse, t[4], (int32_t)frames, g[0], g[1], g[2], g[3], g[4], ws, bytes, s);
      return group ? lib.group_bwd(cache, t[0], t[1], t[2], t[3], lse, t[4], (int32_t)frames, (int32_t)group, g[0], g[1], g[2], ws, bytes, s)
                   : lib.chunk_bwd(cache, t[0], t[1], t[2], t[3], lse, t[4], (int32_t)frames, g[0], g[1], g[2], ws, bytes, s);
    });
  });
}

// (v_theta, v_old, v_ref, target, advantage, kl_mask, a_max, beta, lambda_kl, loss, grad, workspace)
PyObject* loss(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 12) return nullptr;
    Reader r;
    const at::Tensor* const x = r.plain(a[0]);
    if (!x || x->dim() < 1 || !x->is_contiguous()) return nullptr;
    const at::ScalarType type = x->scalar_type();
    const int64_t numel = x->numel(), samples = x->size(0);
    if ((type != at::kBFloat16 && type != at::kFloat) || numel < 1 || samples > INT32_MAX) return nullptr;
    const void* t[4] = {x->data_ptr()};
    for (int i = 1; i < 4; ++i) {
      const at::Tensor* const y = r.plain(a[i]);
      if (!y || y->sizes() != x->sizes() || y->scalar_type() != type || !y->is_contiguous()) return nullptr;
      t[i] = y->data_ptr();
    }
    void* const advantage = r.of_type(a[4], at::kFloat, samples);
    void* const mask = r.of_type(a[5], at::kInt, samples);
    const float a_max = r.number(a[6]), beta = r.number(a[7]), lambda = r.number(a[8]);
    const at::Tensor* const l = r.plain(a[9]);
    if (!l || l->scalar_type() != at::kFloat || l->numel() < 3 || !l->is_contiguous()) return nullptr;
    void* const to = l->data_ptr();
    void* const grad = r.of_type(a[10], at::kFloat, numel);
    size_t bytes = 0, need = 0;
    void* const ws = r.workspace(a[11], &bytes);
    if (!r.ok || lib.loss_workspace_bytes((int32_t)samples, numel / samples, &need) != ASTRO_OK) return nullptr;
    return run([&](void* s) {
      return lib.loss(t[0], t[1], t[2], t[3], (const float*)advantage, (const int32_t*)mask, (int32_t)samples, numel / samples,
                      type == at::kBFloat16 ? ASTRO_BF16 : ASTRO_F32, a_max, beta, lambda, (float*)to, (float*)grad, ws, bytes, s);
    });
  });
}

// the addresses of Library's functions, in its order
PyObject* bind(PyObject*, PyObject* addresses) {
  constexpr Py_ssize_t kFunctions = sizeof(Library) / sizeof(void*);
  if (!PyTuple_CheckExact(addresses) || PyTuple_GET_SIZE(addresses) != kFunctions) {
    PyErr_SetString(PyExc_TypeError, "bind: a tuple of function addresses");
    return nullptr;
  }
  void* at[kFunctions];
  for (Py_ssize_t i = 0; i < kFunctions; ++i) at[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
  if (PyErr_Occurred()) return nullptr;
  std::memcpy(&lib, at, sizeof(lib));
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_O, nullptr},
    {"append", (PyCFunction)(void (*)(void))append, METH_FASTCALL, nullptr},
    {"fwd", (PyCFunction)(void (*)(void))fwd, METH_FASTCALL, nullptr},
    {"bwd", (PyCFunction)(void (*)(void))bwd, METH_FASTCALL, nullptr},
    {"loss", (PyCFunction)(void (*)(void))loss, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding_native() {
  PyObject* const m = PyModule_Create(&module);
  // the torch whose tensors this file's headers describe: binding.py binds no other's
  if (m && PyModule_AddStringConstant(m, "built_for_torch", BUILT_FOR_TORCH) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
