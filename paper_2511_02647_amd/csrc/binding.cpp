// CPython side of the library: turns the Python arguments of an entry point into the C ABI's
// (include/fedattn.h) and calls it with the interpreter lock released.  A ctypes call took 6-7 us
// of host time per attention call for this (10.6 of 14.9 us at the smallest sizes, where the
// kernels are shorter than that); here it is about one.
//
// bind(addresses, ...) hands over the entry points of the loaded library; every other function takes
// its arguments by position (the Python wrappers hold names and defaults) and returns the status
// code.  Tensors are asked for is_cuda, is_contiguous() and data_ptr(), host arrays come through the
// buffer protocol; `as_i32` (Python) converts what is not an int32 vector already.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <string.h>

#include "fedattn.h"

namespace {

PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_nbytes, *s_numel, *s_cuda_stream;
PyObject *g_params_type, *g_as_i32, *g_raw_stream, *g_get_device;   // set by bind()

decltype(&fedattn_prefill) f_prefill;
decltype(&fedattn_prefill_sync_local_kv) f_prefill_sync_local_kv;
decltype(&fedattn_prefill_blocks) f_prefill_blocks;
decltype(&fedattn_decode_blocks) f_decode_blocks;
decltype(&fedattn_decode_blocks_fused) f_decode_blocks_fused;
decltype(&fedattn_decode_static) f_decode_static;
decltype(&fedattn_aggregate_kv) f_aggregate_kv;
decltype(&fedattn_rmsnorm) f_rmsnorm;
decltype(&fedattn_rope_split_qkv) f_rope_split_qkv;
decltype(&fedattn_swiglu) f_swiglu;
decltype(&fedattn_residual_add) f_residual_add;
decltype(&fedattn_residual_add_rmsnorm) f_residual_add_rmsnorm;

// The arguments of one call, read one after the other; the first failure leaves `ok` false with the
// Python error set.
struct Args {
  PyObject* const* v;
  Py_ssize_t n, at = 0;
  bool ok = true;
  Py_buffer held[5];
  PyObject* converted[5];
  int n_held = 0;

  Args(PyObject* const* v_, Py_ssize_t n_, Py_ssize_t want) : v(v_), n(n_) {
    if (n != want) {
      PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
      ok = false;
    }
  }
  ~Args() {
    for (int i = 0; i < n_held; ++i) {
      PyBuffer_Release(&held[i]);
      Py_XDECREF(converted[i]);
    }
  }
  Args(const Args&) = delete;
  Args& operator=(const Args&) = delete;

  PyObject* next() { return v[at++]; }

  int64_t integer() {
    PyObject* o = next();
    if (!ok) return 0;
    PyObject* idx = PyNumber_Long(o);
    const int64_t x = idx ? (int64_t)PyLong_AsUnsignedLongLongMask(idx) : -1;   // what does not fit is cut off
    Py_XDECREF(idx);
    if (x == -1 && PyErr_Occurred()) ok = false;
    return x;
  }
  double real() {
    PyObject* o = next();
    if (!ok) return 0.0;
    PyObject* num = PyNumber_Float(o);
    const double x = num ? PyFloat_AsDouble(num) : -1.0;
    Py_XDECREF(num);
    if (x == -1.0 && PyErr_Occurred()) ok = false;
    return x;
  }

  // a buffer of the object, held until the call is over
  Py_buffer* hold(PyObject* o, PyObject* owned) {
    Py_buffer* b = &held[n_held];
    if (PyObject_GetBuffer(o, b, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) {
      Py_XDECREF(owned);
      ok = false;
      return nullptr;
    }
    converted[n_held++] = owned;
    return b;
  }

  const fedattn_params* params() {
    PyObject* o = next();
    if (!ok) return nullptr;
    Py_buffer* b = nullptr;
    if (PyObject_TypeCheck(o, (PyTypeObject*)g_params_type)) {
      b = hold(o, nullptr);
    } else {
      PyErr_SetString(PyExc_TypeError, "params must be a fedattn_params");
      ok = false;
    }
    return ok ? static_cast<const fedattn_params*>(b->buf) : nullptr;
  }

  // a host vector of int32; its length in *len
  const int32_t* vec(const char* name, Py_ssize_t* len, bool optional = false) {
    PyObject* o = next();
    *len = -1;
    if (!ok || (optional && o == Py_None)) return nullptr;
    if (PyObject_CheckBuffer(o)) {
      Py_buffer* b = &held[n_held];
      if (PyObject_GetBuffer(o, b, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) == 0) {
        if (b->ndim == 1 && b->itemsize == 4 && b->format && !strcmp(b->format, "i")) {
          converted[n_held++] = nullptr;
          *len = b->shape[0];
          return static_cast<const int32_t*>(b->buf);
        }
        PyBuffer_Release(b);
      } else {
        PyErr_Clear();
      }
    }
    PyObject* arr = PyObject_CallFunction(g_as_i32, "Os", o, name);
    if (!arr) {
      ok = false;
      return nullptr;
    }
    Py_buffer* b = hold(arr, arr);
    if (!b) return nullptr;
    *len = b->shape[0];
    return static_cast<const int32_t*>(b->buf);
  }

  static bool truthy(PyObject* r) {   // consumes r; false also when r is null
    const int t = r ? PyObject_IsTrue(r) : 0;
    Py_XDECREF(r);
    return t == 1;
  }
  void* address(PyObject* o) {
    PyObject* p = PyObject_CallMethodNoArgs(o, s_data_ptr);
    void* x = p ? PyLong_AsVoidPtr(p) : nullptr;
    Py_XDECREF(p);
    if (PyErr_Occurred()) ok = false;
    return x;
  }
  // a device tensor's address; None is NULL, which the library accepts or rejects by its own rules
  void* tensor(const char* name, size_t* bytes = nullptr) {
    PyObject* o = next();
    if (!ok || o == Py_None) return nullptr;
    if (!truthy(PyObject_GetAttr(o, s_is_cuda))) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_TypeError, "%s must be a device tensor", name);
      ok = false;
      return nullptr;
    }
    if (!truthy(PyObject_CallMethodNoArgs(o, s_is_contiguous))) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_TypeError, "%s must be contiguous", name);
      ok = false;
      return nullptr;
    }
    if (bytes) {
      PyObject* nb = PyObject_GetAttr(o, s_nbytes);
      *bytes = nb ? PyLong_AsSize_t(nb) : 0;
      Py_XDECREF(nb);
      if (PyErr_Occurred()) {
        ok = false;
        return nullptr;
      }
    }
    return address(o);
  }
  void* workspace(size_t* bytes) {
    *bytes = 0;
    return tensor("workspace", bytes);
  }
  // device pointers of the participants' matrices; absent and empty ones are NULL
  void locals(const char* name, int n_part, const void** out) {
    PyObject* seq = next();
    for (int i = 0; ok && i < n_part; ++i) {
      PyObject* t = PySequence_GetItem(seq, i);
      if (!t) {
        ok = false;
        return;
      }
      out[i] = nullptr;
      if (t != Py_None) {
        PyObject* cnt = PyObject_CallMethodNoArgs(t, s_numel);
        const bool some = truthy(cnt);
        if (PyErr_Occurred()) {
          ok = false;
        } else if (some) {
          const bool fits = truthy(PyObject_GetAttr(t, s_is_cuda)) && truthy(PyObject_CallMethodNoArgs(t, s_is_contiguous));
          if (fits) {
            out[i] = address(t);
          } else {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_TypeError, "%s[%d] must be a contiguous device tensor", name, i);
            ok = false;
          }
        }
      }
      Py_DECREF(t);
    }
  }
  Py_ssize_t length(Py_ssize_t at_arg) {
    if (!ok) return -1;
    const Py_ssize_t l = PySequence_Size(v[at_arg]);
    if (l < 0) ok = false;
    return l;
  }
  void* stream() {
    PyObject* o = next();
    if (!ok) return nullptr;
    PyObject* h = nullptr;
    if (o == Py_None) {   // the current stream of the current device
      PyObject* dev = PyObject_CallNoArgs(g_get_device);
      h = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
      Py_XDECREF(dev);
    } else {
      h = PyObject_GetAttr(o, s_cuda_stream);
    }
    void* x = h ? PyLong_AsVoidPtr(h) : nullptr;
    Py_XDECREF(h);
    if (PyErr_Occurred()) ok = false;
    return x;
  }
  bool fail(const char* msg) {
    if (ok) PyErr_SetString(PyExc_ValueError, msg);
    ok = false;
    return false;
  }
};

template <typename F>
PyObject* finish(Args& a, F&& call) {
  if (!a.ok) return nullptr;
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = (int)call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

PyObject* py_prefill(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 12);
  if (!a.ok) return nullptr;
  Py_ssize_t ns;
  size_t wsb;
  const fedattn_params* p = a.params();
  const int32_t block = (int32_t)a.integer();
  const void *q = a.tensor("q"), *k = a.tensor("k"), *vv = a.tensor("v");
  void* out = a.tensor("out");
  const int32_t* seg = a.vec("seg_offsets", &ns);
  if (a.ok && ns != p->n_participants + 1) a.fail("seg_offsets must have n_participants + 1 entries");
  const uint8_t* keep = (const uint8_t*)a.tensor("keep_chunks");
  const int32_t chunk = (int32_t)a.integer(), over = (int32_t)a.integer();
  void* ws = a.workspace(&wsb);
  void* st = a.stream();
  return finish(a, [&] { return f_prefill(p, block, q, k, vv, out, seg, keep, chunk, over, ws, wsb, st); });
}

PyObject* py_prefill_sync_local_kv(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 10);
  if (!a.ok) return nullptr;
  Py_ssize_t ns;
  size_t wsb;
  const void *kl[FEDATTN_MAX_PARTICIPANTS], *vl[FEDATTN_MAX_PARTICIPANTS];
  const fedattn_params* p = a.params();
  const Py_ssize_t nk = a.length(2), nv = a.length(3);
  const int N = a.ok ? p->n_participants : 0;
  a.at = 5;
  const int32_t* seg = a.vec("seg_offsets", &ns);
  if (a.ok && (ns != N + 1 || nk != N || nv != N)) a.fail("k_local / v_local / seg_offsets have the wrong length");
  const int n_ptrs = N < 0 || N > FEDATTN_MAX_PARTICIPANTS ? 0 : N;   // the library rejects such a count
  a.at = 1;
  const void* q = a.tensor("q");
  a.locals("k_local", n_ptrs, kl);
  a.locals("v_local", n_ptrs, vl);
  void* out = a.tensor("out");
  a.at = 6;
  const uint8_t* keep = (const uint8_t*)a.tensor("keep_chunks");
  const int32_t chunk = (int32_t)a.integer();
  void* ws = a.workspace(&wsb);
  void* st = a.stream();
  return finish(a, [&] { return f_prefill_sync_local_kv(p, q, kl, vl, out, seg, keep, chunk, ws, wsb, st); });
}

PyObject* py_prefill_blocks(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 11);
  if (!a.ok) return nullptr;
  Py_ssize_t ns;
  const fedattn_params* p = a.params();
  const int32_t block = (int32_t)a.integer(), count = (int32_t)a.integer();
  const void *q = a.tensor("q"), *k = a.tensor("k"), *vv = a.tensor("v");
  void* out = a.tensor("out");
  const int64_t qs = a.integer(), ks = a.integer();
  const int32_t* seg = a.vec("seg_offsets", &ns);
  if (a.ok && ns != p->n_participants + 1) a.fail("seg_offsets must have n_participants + 1 entries");
  void* st = a.stream();
  return finish(a, [&] { return f_prefill_blocks(p, block, count, q, k, vv, out, qs, ks, seg, st); });
}

// the three length vectors of a decode call
struct DecodeLens {
  const int32_t *seg, *lens, *remote;
  explicit DecodeLens(Args& a, const fedattn_params* p) {
    Py_ssize_t ns, nl, nr;
    seg = a.vec("seg_offsets", &ns);
    lens = a.vec("seg_lens", &nl);
    if (a.ok && (ns != p->n_participants + 1 || nl != p->n_participants)) a.fail("seg_offsets / seg_lens have the wrong length");
    remote = a.vec("remote_lens", &nr, true);
    if (a.ok && remote && nr != p->n_participants) a.fail("remote_lens has the wrong length");
  }
};

// (params, block0, n_blocks, q, k, v, out, q_stride, cache_stride, seg, lens, remote, override, workspace, stream, fused)
PyObject* py_decode_blocks(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 16);
  if (!a.ok) return nullptr;
  size_t wsb;
  const fedattn_params* p = a.params();
  const int32_t block = (int32_t)a.integer(), count = (int32_t)a.integer();
  const void *q = a.tensor("q"), *k = a.tensor("k_cache"), *vv = a.tensor("v_cache");
  void* out = a.tensor("out");
  const int64_t qs = a.integer(), cs = a.integer();
  const DecodeLens l(a, p);
  const int32_t over = (int32_t)a.integer();
  void* ws = a.workspace(&wsb);
  void* st = a.stream();
  const auto fn = a.ok && a.integer() ? f_decode_blocks_fused : f_decode_blocks;
  return finish(a, [&] { return fn(p, block, count, q, k, vv, out, qs, cs, l.seg, l.lens, l.remote, over, ws, wsb, st); });
}

PyObject* py_decode_static(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 11);
  if (!a.ok) return nullptr;
  const fedattn_params* p = a.params();
  const int32_t block = (int32_t)a.integer();
  const void *q = a.tensor("q"), *k = a.tensor("k_cache"), *vv = a.tensor("v_cache");
  void* out = a.tensor("out");
  const DecodeLens l(a, p);
  const int32_t over = (int32_t)a.integer();
  void* st = a.stream();
  return finish(a, [&] { return f_decode_static(p, block, q, k, vv, out, l.seg, l.lens, l.remote, over, st); });
}

PyObject* py_aggregate_kv(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 7);
  if (!a.ok) return nullptr;
  Py_ssize_t ns;
  const void *kl[FEDATTN_MAX_PARTICIPANTS], *vl[FEDATTN_MAX_PARTICIPANTS];
  const fedattn_params* p = a.params();
  const Py_ssize_t nk = a.length(1), nv = a.length(2);
  const int N = a.ok ? p->n_participants : 0;
  a.at = 3;
  const int32_t* seg = a.vec("seg_offsets", &ns);
  if (a.ok && (ns != N + 1 || nk != N || nv != N)) a.fail("k_local / v_local / seg_offsets have the wrong length");
  const int n_ptrs = N < 0 || N > FEDATTN_MAX_PARTICIPANTS ? 0 : N;
  a.at = 1;
  a.locals("k_local", n_ptrs, kl);
  a.locals("v_local", n_ptrs, vl);
  a.at = 4;
  void *kg = a.tensor("k_global"), *vg = a.tensor("v_global");
  void* st = a.stream();
  return finish(a, [&] { return f_aggregate_kv(p, kl, vl, seg, kg, vg, st); });
}

// (x, y or None, out, rows, d_model, eps, stream)
PyObject* py_rmsnorm(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 7);
  if (!a.ok) return nullptr;
  float* x = (float*)a.tensor("x");
  const bool add = v[1] != Py_None;
  const void* y = a.tensor("y");
  void* out = a.tensor("out");
  const int64_t rows = a.integer();
  const int32_t d = (int32_t)a.integer();
  const float eps = (float)a.real();
  void* st = a.stream();
  return finish(a, [&] { return add ? f_residual_add_rmsnorm(x, y, out, rows, d, eps, st) : f_rmsnorm(x, out, rows, d, eps, st); });
}

PyObject* py_rope_split_qkv(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 11);
  if (!a.ok) return nullptr;
  const void* qkv = a.tensor("qkv");
  const int32_t* pos = (const int32_t*)a.tensor("pos");
  void *q = a.tensor("q"), *k = a.tensor("k"), *vv = a.tensor("v");
  const int64_t t = a.integer();
  const int32_t hq = (int32_t)a.integer(), hkv = (int32_t)a.integer(), d = (int32_t)a.integer();
  const float theta = (float)a.real();
  void* st = a.stream();
  return finish(a, [&] { return f_rope_split_qkv(qkv, pos, q, k, vv, t, hq, hkv, d, theta, st); });
}

PyObject* py_swiglu(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 5);
  if (!a.ok) return nullptr;
  const void* gu = a.tensor("gate_up");
  void* out = a.tensor("out");
  const int64_t rows = a.integer();
  const int32_t hidden = (int32_t)a.integer();
  void* st = a.stream();
  return finish(a, [&] { return f_swiglu(gu, out, rows, hidden, st); });
}

PyObject* py_residual_add(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Args a(v, n, 4);
  if (!a.ok) return nullptr;
  float* x = (float*)a.tensor("x");
  const void* y = a.tensor("y");
  const int64_t cnt = a.integer();
  void* st = a.stream();
  return finish(a, [&] { return f_residual_add(x, y, cnt, st); });
}

// bind(addresses: dict name -> int, params_type: the ctypes structure, as_i32, raw_stream, get_device)
PyObject* py_bind(PyObject*, PyObject* args) {
  PyObject *dict, *type, *as_i32, *raw, *dev;
  if (!PyArg_ParseTuple(args, "O!O!OOO", &PyDict_Type, &dict, &PyType_Type, &type, &as_i32, &raw, &dev)) return nullptr;
#define BIND(name)                                                             \
  {                                                                            \
    PyObject* x = PyDict_GetItemString(dict, "fedattn_" #name);                \
    if (!x) return PyErr_Format(PyExc_KeyError, "fedattn_" #name);             \
    f_##name = reinterpret_cast<decltype(f_##name)>(PyLong_AsVoidPtr(x));      \
    if (PyErr_Occurred()) return nullptr;                                      \
  }
  BIND(prefill) BIND(prefill_sync_local_kv) BIND(prefill_blocks) BIND(decode_blocks) BIND(decode_blocks_fused)
  BIND(decode_static) BIND(aggregate_kv) BIND(rmsnorm) BIND(rope_split_qkv) BIND(swiglu) BIND(residual_add)
  BIND(residual_add_rmsnorm)
#undef BIND
  Py_INCREF(type); Py_XSETREF(g_params_type, type);
  Py_INCREF(as_i32); Py_XSETREF(g_as_i32, as_i32);
  Py_INCREF(raw); Py_XSETREF(g_raw_stream, raw);
  Py_INCREF(dev); Py_XSETREF(g_get_device, dev);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(prefill), FAST(prefill_sync_local_kv), FAST(prefill_blocks), FAST(decode_blocks),
                         FAST(decode_static), FAST(aggregate_kv), FAST(rmsnorm), FAST(rope_split_qkv), FAST(swiglu),
                         FAST(residual_add), {"bind", py_bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Argument marshalling of the FedAttn library.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_nbytes = PyUnicode_InternFromString("nbytes");
  s_numel = PyUnicode_InternFromString("numel");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  return PyModule_Create(&module);
}
