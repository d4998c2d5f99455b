// Calls the three entry points that a decoder makes per layer and step with tensors straight from Python.  ctypes converts fourteen
// arguments, eight of them fetched by a Python function each, in 2.2 us, as much as a kernel launch; this takes 0.9.  The functions
// are given by address, so that they are those of the library that the binding has loaded.  Each returns what the entry point does;
// block_step the state that it executed where that succeeded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <initializer_list>

#include "sdllm.h"

namespace {

PyObject *s_data_ptr, *s_numel, *s_element_size;

// Arguments in order; the first that cannot be had leaves an exception and zeroes after it.
struct Args {
  PyObject* const* at;
  bool ok = true;

  void* address(PyObject* number) {
    void* p = ok ? PyLong_AsVoidPtr(number) : nullptr;
    if (ok && !p && PyErr_Occurred()) ok = false;
    return p;
  }
  void* address() { return address(*at++); }
  long number() {
    const long v = ok ? PyLong_AsLong(*at) : 0;
    if (ok && v == -1 && PyErr_Occurred()) ok = false;
    ++at;
    return v;
  }
  // a tensor's memory, null for None
  void* tensor() {
    PyObject* t = *at++;
    if (!ok || t == Py_None) return nullptr;
    PyObject* p = PyObject_CallMethodNoArgs(t, s_data_ptr);
    if (!p) { ok = false; return nullptr; }
    void* v = address(p);
    Py_DECREF(p);
    return v;
  }
  // bytes of the tensor that is next, 0 for None
  size_t bytes() {
    if (!ok || *at == Py_None) return 0;
    size_t n = 1;
    for (PyObject* name : {s_numel, s_element_size}) {
      PyObject* v = PyObject_CallMethodNoArgs(*at, name);
      if (!v) { ok = false; return 0; }
      n *= PyLong_AsSize_t(v);
      Py_DECREF(v);
      if (PyErr_Occurred()) { ok = false; return 0; }
    }
    return n;
  }
  void strides(int64_t (&s)[3]) {
    PyObject* t = *at++;
    for (int i = 0; i < 3; ++i) {
      s[i] = 0;
      if (!ok) continue;
      if (!PyTuple_Check(t) || PyTuple_GET_SIZE(t) != 3) { PyErr_SetString(PyExc_TypeError, "three strides"); ok = false; continue; }
      s[i] = PyLong_AsLongLong(PyTuple_GET_ITEM(t, i));
      if (s[i] == -1 && PyErr_Occurred()) ok = false;
    }
  }
};

bool count_is(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments, not %zd", want, n);
  return false;
}

PyObject* block_step(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count_is(n, 13)) return nullptr;
  Args a{args};
  const auto f = reinterpret_cast<decltype(&sdllm_block_step)>(a.address());
  const auto* shape = static_cast<const sdllm_shape_t*>(a.address());
  const int32_t step = (int32_t)a.number(), delay = (int32_t)a.number();
  void *q = a.tensor(), *k = a.tensor(), *v = a.tensor(), *idx = a.tensor(), *kc = a.tensor(), *vc = a.tensor(), *out = a.tensor();
  const size_t ws_bytes = a.bytes();
  void *ws = a.tensor(), *stream = a.address();
  if (!a.ok) return nullptr;
  int32_t status, state = -1;
  Py_BEGIN_ALLOW_THREADS
  status = f(shape, step, delay, q, k, v, static_cast<int32_t*>(idx), kc, vc, out, ws, ws_bytes, stream, &state);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status == SDLLM_OK ? state : status);
}

PyObject* sparse_attn(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count_is(n, 11)) return nullptr;
  Args a{args};
  const auto f = reinterpret_cast<decltype(&sdllm_sparse_attn)>(a.address());
  const auto* shape = static_cast<const sdllm_shape_t*>(a.address());
  void *q = a.tensor(), *kc = a.tensor(), *vc = a.tensor();
  const int32_t n_cached = (int32_t)a.number();
  void *kb = a.tensor(), *vb = a.tensor(), *out = a.tensor();
  const size_t ws_bytes = a.bytes();
  void *ws = a.tensor(), *stream = a.address();
  if (!a.ok) return nullptr;
  int32_t status;
  Py_BEGIN_ALLOW_THREADS
  status = f(shape, q, kc, vc, n_cached, kb, vb, out, ws, ws_bytes, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

PyObject* dense_attn(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count_is(n, 9)) return nullptr;
  Args a{args};
  const auto f = reinterpret_cast<decltype(&sdllm_dense_attn)>(a.address());
  const auto* shape = static_cast<const sdllm_shape_t*>(a.address());
  int64_t q_stride[3], out_stride[3];
  void* q = a.tensor();
  a.strides(q_stride);
  void *k = a.tensor(), *v = a.tensor(), *out = a.tensor();
  a.strides(out_stride);
  void* stream = a.address();
  if (!a.ok) return nullptr;
  int32_t status;
  Py_BEGIN_ALLOW_THREADS
  status = f(shape, q, q_stride, k, v, out, out_stride, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

template <class F>
PyCFunction fast(F* f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef methods[] = {
    {"block_step", fast(block_step), METH_FASTCALL, "function, shape, step, delay, q, k, v, idx, k_cache, v_cache, out, ws, stream"},
    {"sparse_attn", fast(sparse_attn), METH_FASTCALL, "function, shape, q, k_cache, v_cache, n_cached, k, v, out, ws, stream"},
    {"dense_attn", fast(dense_attn), METH_FASTCALL, "function, shape, q, q strides, k, v, out, out strides, stream"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall() {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  return s_data_ptr && s_numel && s_element_size ? PyModule_Create(&module) : nullptr;
}
