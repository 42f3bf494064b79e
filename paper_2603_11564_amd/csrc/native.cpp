// The calls of binding.py as native code (the extension module _native): tensors become pointers, the current torch stream a hipStream_t, and the
// library's function is called without the interpreter's lock.  Nothing is computed here, and nothing of a call is kept.
//
// Beside the library's own 2.4 to 2.8 us (a launch; two 5.3 to 6.0) a call took the host 1.7 to 2.0 us through ctypes and takes 0.7 to 0.8 here,
// which is what small kernels wait for: projection of one layer 1024 wide with its pseudo tokens 13.8 -> 12.4 us a pass, score call of one layer and
// 1024 keys with its rotation 11.4 -> 9.2 of host time.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

#include "dapq.h"

namespace {

PyObject *g_resolver = nullptr, *g_stream = nullptr, *g_device = nullptr;  // see stream_of
PyTypeObject *g_shape = nullptr, *g_qproj = nullptr;                       // the descriptors' classes
PyObject* g_other_way = nullptr;                                           // see other_way
PyObject *g_data_ptr, *g_numel, *g_element_size, *g_cuda_stream;           // interned names

// Every converter returns false with a Python error set.
bool pointer_of(PyObject* tensor, void** out) {
  *out = nullptr;
  if (tensor == Py_None) return true;
  PyObject* v = PyObject_CallMethodNoArgs(tensor, g_data_ptr);
  if (v == nullptr) return false;
  *out = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(v));
  Py_DECREF(v);
  return PyErr_Occurred() == nullptr;
}
bool bytes_of(PyObject* tensor, size_t* out) {
  *out = 0;
  if (tensor == Py_None) return true;
  PyObject *n = PyObject_CallMethodNoArgs(tensor, g_numel), *e = n ? PyObject_CallMethodNoArgs(tensor, g_element_size) : nullptr;
  if (e != nullptr) *out = (size_t)(PyLong_AsUnsignedLongLongMask(n) * PyLong_AsUnsignedLongLongMask(e));
  Py_XDECREF(n);
  Py_XDECREF(e);
  return PyErr_Occurred() == nullptr;
}
bool int_of(PyObject* v, int64_t* out) {
  if (PyFloat_Check(v)) {
    PyErr_SetString(PyExc_TypeError, "int expected instead of float");
    return false;
  }
  *out = (int64_t)PyLong_AsUnsignedLongLongMask(v);
  return PyErr_Occurred() == nullptr;
}
// None: the current torch stream.  The resolver gives the function of its handle and the one of the current device (or None, and the first
// takes no argument), once, when the first call needs them: torch initialises the device then.
bool stream_of(PyObject* s, void** out) {
  *out = nullptr;
  PyObject* v = nullptr;
  if (s != Py_None) {
    if (PyLong_Check(s)) {
      v = s;
      Py_INCREF(v);
    } else {
      v = PyObject_GetAttr(s, g_cuda_stream);
    }
  } else {
    if (g_stream == nullptr) {
      PyObject* pair = PyObject_CallNoArgs(g_resolver);
      if (pair == nullptr) return false;
      PyObject *stream, *device;
      if (!PyArg_ParseTuple(pair, "OO", &stream, &device)) {
        Py_DECREF(pair);
        return false;
      }
      Py_INCREF(stream);
      Py_INCREF(device);
      Py_DECREF(pair);
      Py_XSETREF(g_device, device);
      Py_XSETREF(g_stream, stream);
    }
    PyObject *stream = g_stream, *device = g_device;  // (kept for the calls, during which another thread may bind anew)
    Py_INCREF(stream);
    Py_INCREF(device);
    if (device == Py_None) {
      v = PyObject_CallNoArgs(stream);
    } else if (PyObject* d = PyObject_CallNoArgs(device)) {
      v = PyObject_CallOneArg(stream, d);
      Py_DECREF(d);
    }
    Py_DECREF(device);
    Py_DECREF(stream);
  }
  if (v == nullptr) return false;
  *out = reinterpret_cast<void*>((uintptr_t)PyLong_AsUnsignedLongLongMask(v));
  Py_DECREF(v);
  return PyErr_Occurred() == nullptr;
}
// A copy of a descriptor (a ctypes structure of its own class).
PyTypeObject* class_of(const dapq_shape*) { return g_shape; }
PyTypeObject* class_of(const dapq_qproj*) { return g_qproj; }
template <typename T>
bool struct_of(PyObject* v, T* out) {
  if (class_of(out) == nullptr || !PyObject_TypeCheck(v, class_of(out))) {
    PyErr_Format(PyExc_TypeError, "descriptor expected instead of %s", Py_TYPE(v)->tp_name);
    return false;
  }
  Py_buffer b;
  if (PyObject_GetBuffer(v, &b, PyBUF_SIMPLE) != 0) return false;
  const bool ok = b.len == (Py_ssize_t)sizeof(T);
  if (ok) *out = *static_cast<const T*>(b.buf);
  else PyErr_Format(PyExc_TypeError, "descriptor of %zd bytes, %zd expected", b.len, (Py_ssize_t)sizeof(T));
  PyBuffer_Release(&b);
  return ok;
}
bool count_is(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", n, want);
  return false;
}

// The library's functions, by the order of `kNames`; binding.py hands over their addresses.
struct Calls {
  decltype(&dapq_rope_apply) rope_apply;
  decltype(&dapq_score) score;
  decltype(&dapq_score_static) score_static;
  decltype(&dapq_score_stats) score_stats;
  decltype(&dapq_score_accumulate) score_accumulate;
  decltype(&dapq_score_stats_extend) score_stats_extend;
  decltype(&dapq_pool) pool;
  decltype(&dapq_topk) topk;
  decltype(&dapq_pool_topk) pool_topk;
  decltype(&dapq_gather) gather;
  decltype(&dapq_recall) recall;
  decltype(&dapq_decode_attention) decode_attention;
  decltype(&dapq_pseudo_tokens) pseudo_tokens;
  decltype(&dapq_pseudo_queries) pseudo_queries;
};
const char* const kNames[] = {"dapq_rope_apply", "dapq_score", "dapq_score_static", "dapq_score_stats", "dapq_score_accumulate",
                              "dapq_score_stats_extend", "dapq_pool", "dapq_topk", "dapq_pool_topk", "dapq_gather", "dapq_recall",
                              "dapq_decode_attention", "dapq_pseudo_tokens", "dapq_pseudo_queries"};
constexpr int kCalls = (int)(sizeof(kNames) / sizeof(kNames[0]));
static_assert(sizeof(Calls) == kCalls * sizeof(void*), "a name for every function");
Calls g_calls = {};

// (addresses by name, resolver of the current stream, Shape, Qproj, the way through ctypes)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (!count_is(n, 5)) return nullptr;
  if (!PyType_Check(a[2]) || !PyType_Check(a[3])) return PyErr_Format(PyExc_TypeError, "classes expected");
  void* at[kCalls];
  for (int i = 0; i < kCalls; ++i) {
    PyObject* v = PyDict_Check(a[0]) ? PyDict_GetItemString(a[0], kNames[i]) : nullptr;
    if (v == nullptr) return PyErr_Format(PyExc_KeyError, "%s", kNames[i]);
    at[i] = PyLong_AsVoidPtr(v);
    if (PyErr_Occurred()) return nullptr;
  }
  __builtin_memcpy(&g_calls, at, sizeof(at));
  Py_INCREF(a[1]);
  Py_XSETREF(g_resolver, a[1]);
  Py_INCREF(a[2]);
  Py_XSETREF(g_shape, reinterpret_cast<PyTypeObject*>(a[2]));
  Py_INCREF(a[3]);
  Py_XSETREF(g_qproj, reinterpret_cast<PyTypeObject*>(a[3]));
  Py_INCREF(a[4]);
  Py_XSETREF(g_other_way, a[4]);
  Py_CLEAR(g_stream);
  Py_CLEAR(g_device);
  Py_RETURN_NONE;
}

// A call with an argument of a kind that is not converted here (a number or an address as a ctypes object, a descriptor with more fields, a handle
// of None): ctypes takes it, or refuses it.  With another error than a TypeError set, that one stays.
PyObject* other_way(const char* name, PyObject* const* a, Py_ssize_t n) {
  if (!PyErr_ExceptionMatches(PyExc_TypeError)) return nullptr;
  PyErr_Clear();
  PyObject* all = PyTuple_New(n + 1);
  PyObject* first = all ? PyUnicode_FromString(name) : nullptr;
  if (first == nullptr) {
    Py_XDECREF(all);
    return nullptr;
  }
  PyTuple_SET_ITEM(all, 0, first);
  for (Py_ssize_t i = 0; i < n; ++i) {
    Py_INCREF(a[i]);
    PyTuple_SET_ITEM(all, i + 1, a[i]);
  }
  PyObject* rc = g_other_way ? PyObject_CallObject(g_other_way, all) : PyErr_Format(PyExc_RuntimeError, "not bound to the library");
  Py_DECREF(all);
  return rc;
}

// The call itself, without the interpreter's lock (a full queue makes a launch wait); its return code as a Python number.
template <typename F>
PyObject* without_lock(F call) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}
#define P(i) pointer_of(a[i], &p[i])
#define I(i) int_of(a[i], &x[i])
#define FP(i) static_cast<float*>(p[i])
#define IP(i) static_cast<int32_t*>(p[i])
#define I32(i) (int32_t)x[i]
#define ARGS(count)                             \
  if (!count_is(n, count)) return nullptr;      \
  void* p[count] = {};                          \
  int64_t x[count] = {};                        \
  (void)p;                                      \
  (void)x

PyObject* rope_apply(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(11);
  if (!(P(0) && P(1) && P(2) && I(3) && I(4) && I(5) && I(6) && I(7) && I(9) && stream_of(a[10], &p[10]))) return other_way("dapq_rope_apply", a, n);
  const double theta = PyFloat_AsDouble(a[8]);
  if (PyErr_Occurred()) return nullptr;
  return without_lock([&] { return g_calls.rope_apply(p[0], p[1], IP(2), x[3], I32(4), I32(5), x[6], x[7], theta, I32(9), p[10]); });
}
PyObject* score(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(6);
  dapq_shape s;
  size_t bytes;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && P(3) && P(4) && bytes_of(a[4], &bytes) && stream_of(a[5], &p[5]))) return other_way("dapq_score", a, n);
  return without_lock([&] { return g_calls.score(&s, p[1], p[2], FP(3), p[4], bytes, p[5]); });
}
PyObject* score_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(5);
  dapq_shape s;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && P(3) && stream_of(a[4], &p[4]))) return other_way("dapq_score_static", a, n);
  return without_lock([&] { return g_calls.score_static(&s, p[1], p[2], FP(3), p[4]); });
}
PyObject* score_stats(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(6);
  dapq_shape s;
  size_t bytes;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && P(3) && P(4) && bytes_of(a[4], &bytes) && stream_of(a[5], &p[5]))) return other_way("dapq_score_stats", a, n);
  return without_lock([&] { return g_calls.score_stats(&s, p[1], p[2], FP(3), p[4], bytes, p[5]); });
}
PyObject* score_accumulate(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(7);
  dapq_shape s;
  size_t bytes;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && P(3) && P(4) && P(5) && bytes_of(a[5], &bytes) && stream_of(a[6], &p[6]))) return other_way("dapq_score_accumulate", a, n);
  return without_lock([&] { return g_calls.score_accumulate(&s, p[1], p[2], FP(3), FP(4), p[5], bytes, p[6]); });
}
PyObject* score_stats_extend(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(9);
  dapq_shape s;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && I(3) && I(4) && I(5) && I(6) && P(7) && stream_of(a[8], &p[8]))) return other_way("dapq_score_stats_extend", a, n);
  return without_lock([&] { return g_calls.score_stats_extend(&s, p[1], p[2], x[3], x[4], x[5], x[6], FP(7), p[8]); });
}
PyObject* pool(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(5);
  dapq_shape s;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && I(3) && stream_of(a[4], &p[4]))) return other_way("dapq_pool", a, n);
  return without_lock([&] { return g_calls.pool(&s, FP(1), FP(2), I32(3), p[4]); });
}
PyObject* topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(8);
  dapq_shape s;
  size_t bytes;
  if (!(struct_of(a[0], &s) && P(1) && I(2) && P(3) && P(4) && P(5) && P(6) && bytes_of(a[6], &bytes) && stream_of(a[7], &p[7]))) return other_way("dapq_topk", a, n);
  return without_lock([&] { return g_calls.topk(&s, FP(1), I32(2), IP(3), IP(4), IP(5), p[6], bytes, p[7]); });
}
PyObject* pool_topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(10);
  dapq_shape s;
  size_t bytes;
  if (!(struct_of(a[0], &s) && P(1) && I(2) && I(3) && P(4) && P(5) && P(6) && P(7) && P(8) && bytes_of(a[8], &bytes) && stream_of(a[9], &p[9])))
    return other_way("dapq_pool_topk", a, n);
  return without_lock([&] { return g_calls.pool_topk(&s, FP(1), I32(2), I32(3), IP(4), IP(5), IP(6), FP(7), p[8], bytes, p[9]); });
}
PyObject* gather(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(9);
  dapq_shape s;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && P(3) && P(4) && I(5) && P(6) && P(7) && stream_of(a[8], &p[8]))) return other_way("dapq_gather", a, n);
  return without_lock([&] { return g_calls.gather(&s, p[1], p[2], IP(3), IP(4), I32(5), p[6], p[7], p[8]); });
}
PyObject* recall(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(10);
  dapq_shape s;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && I(3) && P(4) && P(5) && I(6) && P(7) && P(8) && stream_of(a[9], &p[9]))) return other_way("dapq_recall", a, n);
  return without_lock([&] { return g_calls.recall(&s, IP(1), IP(2), I32(3), IP(4), IP(5), I32(6), IP(7), FP(8), p[9]); });
}
PyObject* decode_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(8);
  dapq_shape s;
  if (!(struct_of(a[0], &s) && P(1) && P(2) && P(3) && P(4) && I(5) && P(6) && stream_of(a[7], &p[7]))) return other_way("dapq_decode_attention", a, n);
  return without_lock([&] { return g_calls.decode_attention(&s, p[1], p[2], p[3], IP(4), I32(5), FP(6), p[7]); });
}
PyObject* pseudo_tokens(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(6);
  dapq_shape s;
  if (!(struct_of(a[0], &s) && I(1) && I(2) && P(3) && P(4) && stream_of(a[5], &p[5]))) return other_way("dapq_pseudo_tokens", a, n);
  return without_lock([&] { return g_calls.pseudo_tokens(&s, I32(1), I32(2), IP(3), IP(4), p[5]); });
}
PyObject* pseudo_queries(PyObject*, PyObject* const* a, Py_ssize_t n) {
  ARGS(10);
  dapq_qproj d;
  size_t bytes;
  if (!(struct_of(a[0], &d) && P(1) && P(2) && P(3) && P(4) && I(6) && P(7) && P(8) && bytes_of(a[8], &bytes) && stream_of(a[9], &p[9])))
    return other_way("dapq_pseudo_queries", a, n);
  const double theta = PyFloat_AsDouble(a[5]);
  if (PyErr_Occurred()) return nullptr;
  return without_lock([&] { return g_calls.pseudo_queries(&d, p[1], IP(2), p[3], IP(4), theta, I32(6), p[7], p[8], bytes, p[9]); });
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {ENTRY(bind), ENTRY(rope_apply), ENTRY(score), ENTRY(score_static), ENTRY(score_stats), ENTRY(score_accumulate),
                          ENTRY(score_stats_extend), ENTRY(pool), ENTRY(topk), ENTRY(pool_topk), ENTRY(gather), ENTRY(recall),
                          ENTRY(decode_attention), ENTRY(pseudo_tokens), ENTRY(pseudo_queries), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native", "calls of libdapq with torch tensors", -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  g_numel = PyUnicode_InternFromString("numel");
  g_element_size = PyUnicode_InternFromString("element_size");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!g_data_ptr || !g_numel || !g_element_size || !g_cuda_stream) return nullptr;
  return PyModule_Create(&kModule);
}
