// Native call path of the Python binding: the library's entry points as Python functions that take tensors directly.
//
// A decode step passes nineteen arguments.  Turning tensors into addresses in Python and addresses into C values in
// ctypes took 8 us of host time a call, more than the GPU needs for the step of a small model; here the same call costs
// under 1 us.  A pointer argument is a tensor, an integer address, None (NULL) or any object with data_ptr().  Nothing else
// is one: most pointers are device memory, and host memory taken for it (a numpy array, a bytes object) would be read by a
// kernel.  Only a page book, which the library's host functions read, is a writable buffer (the ctypes structure).  The
// argument types come from the declarations in mtla.h.  The addresses of the functions are handed in by the binding
// (bind), which has loaded the library: this module does not link against it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <exception>
#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/mtla.h"

namespace {

// What a call needs beyond its C arguments: storage for structures built from dicts, buffers to release.
struct Hold {
  mtla_layer_weights lw;
  Py_buffer view;
  bool has_view = false;
  ~Hold() {
    if (has_view) PyBuffer_Release(&view);
  }
};

bool address(PyObject* o, void*& out) {
  if (o == Py_None) {
    out = nullptr;
    return true;
  }
  if (THPVariable_Check(o)) {
    out = THPVariable_Unpack(o).data_ptr();
    return true;
  }
  if (PyLong_Check(o)) {
    out = PyLong_AsVoidPtr(o);
    return !(out == nullptr && PyErr_Occurred());
  }
  PyObject* p = PyObject_CallMethod(o, "data_ptr", nullptr);
  if (!p) return false;
  out = PyLong_AsVoidPtr(p);
  Py_DECREF(p);
  return !(out == nullptr && PyErr_Occurred());
}

// A structure of the caller's in host memory, by the buffer protocol (ctypes structures offer it).
bool structure(PyObject* o, size_t bytes, Hold& hold, void*& out) {
  if (o == Py_None) {
    out = nullptr;
    return true;
  }
  if (hold.has_view) {
    PyErr_SetString(PyExc_TypeError, "more than one structure argument");
    return false;
  }
  if (PyObject_GetBuffer(o, &hold.view, PyBUF_WRITABLE) != 0) return false;
  hold.has_view = true;
  if ((size_t)hold.view.len != bytes) {
    PyErr_Format(PyExc_TypeError, "a structure of %zu bytes is needed, the buffer has %zd", bytes, hold.view.len);
    return false;
  }
  out = hold.view.buf;
  return true;
}

// Entry `key` of the mapping d (the layer's weights): one that is required raises KeyError if it is missing.
struct Entry {
  PyObject* o = nullptr;
  ~Entry() { Py_XDECREF(o); }
};
bool entry(PyObject* d, const char* key, bool required, Entry& e) {
  if (required) return (e.o = PyMapping_GetItemString(d, key)) != nullptr;
  if (PyDict_Check(d)) {
    e.o = PyDict_GetItemString(d, key);
    Py_XINCREF(e.o);
    return true;
  }
  return (e.o = PyObject_CallMethod(d, "get", "s", key)) != nullptr;
}

bool weight(PyObject* d, const char* key, bool required, const void*& out) {
  Entry e;
  void* p = nullptr;
  if (!entry(d, key, required, e) || (e.o && !address(e.o, p))) return false;
  out = p;
  return true;
}

bool number(PyObject* d, const char* key, float& out) {
  Entry e;
  if (!entry(d, key, false, e)) return false;
  out = 0.f;
  if (!e.o || (e.o == Py_None && !PyDict_Check(d))) return true;  // absent (None is what another mapping's get returns)
  out = (float)PyFloat_AsDouble(e.o);
  return !PyErr_Occurred();
}

bool layer_weights(PyObject* d, mtla_layer_weights& w) {
  Entry dm;
  if (!weight(d, "w_q", true, w.w_q) || !weight(d, "w_qr", true, w.w_qr) || !weight(d, "w_r", true, w.w_r) ||
      !weight(d, "w_kr", true, w.w_kr) || !weight(d, "w_o", true, w.w_o) || !weight(d, "ln_gamma", false, w.ln_gamma) ||
      !weight(d, "ln_beta", false, w.ln_beta) || !entry(d, "d_model", true, dm) || !number(d, "ln_eps", w.ln_eps) ||
      !number(d, "rope_base", w.rope_base))
    return false;
  w.d_model = (int32_t)PyLong_AsLong(dm.o);
  return !PyErr_Occurred();
}

template <class T>
bool convert(PyObject* o, Hold& hold, T& out) {
  if constexpr (std::is_pointer_v<T>) {
    if constexpr (std::is_same_v<T, const mtla_layer_weights*>) {
      if (!layer_weights(o, hold.lw)) return false;
      out = &hold.lw;
    } else {
      void* p;
      const bool ok = std::is_same_v<T, mtla_page_book*> ? structure(o, sizeof(mtla_page_book), hold, p) : address(o, p);
      if (!ok) return false;
      out = reinterpret_cast<T>(p);
    }
    return true;
  } else {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) return false;
    out = (T)v;
    return true;
  }
}

template <class R, class... A, size_t... I>
PyObject* invoke(R (*fn)(A...), PyObject* const* args, Py_ssize_t n, const char* name, std::index_sequence<I...>) {
  if (!fn) {
    PyErr_Format(PyExc_RuntimeError, "%s: not bound", name);
    return nullptr;
  }
  if (n != (Py_ssize_t)sizeof...(A)) {
    PyErr_Format(PyExc_TypeError, "%s takes %d arguments, %d given", name, (int)sizeof...(A), (int)n);
    return nullptr;
  }
  std::tuple<A...> v{};
  Hold hold;
  try {
    if (!(convert(args[I], hold, std::get<I>(v)) && ...)) return nullptr;
  } catch (const std::exception& e) {  // a tensor without storage
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
  R rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(std::get<I>(v)...);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)rc);
}

// One table row per entry point: its address once bound, and the Python function.
#define ENTRY_POINTS(X)                                                                                              \
  X(mtla_cache_append) X(mtla_decode_attn) X(mtla_decode_step) X(mtla_decode_step_static) X(mtla_cache_append_paged) \
  X(mtla_decode_attn_paged) X(mtla_decode_step_paged) X(mtla_prefill_chunk_attn_paged) X(mtla_prefill_step_paged)    \
  X(mtla_cache_fork_paged) X(mtla_prefill_attn) X(mtla_prefill_chunk_attn) X(mtla_prefill_step) X(mtla_cache_reorder) \
  X(mtla_cache_reorder_from) X(mtla_layer_decode_step) X(mtla_layer_prefill) X(mtla_pages_reserve) X(mtla_pages_fork)

#define DEFINE(NAME)                                                                                            \
  decltype(&NAME) p_##NAME = nullptr;                                                                           \
  template <class R, class... A>                                                                                \
  PyObject* go_##NAME(R (*fn)(A...), PyObject* const* args, Py_ssize_t n) {                                     \
    return invoke(fn, args, n, #NAME, std::index_sequence_for<A...>());                                         \
  }                                                                                                             \
  PyObject* py_##NAME(PyObject*, PyObject* const* args, Py_ssize_t n) { return go_##NAME(p_##NAME, args, n); }
ENTRY_POINTS(DEFINE)
#undef DEFINE

// bind(name, address)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 2) return PyErr_Format(PyExc_TypeError, "bind(name, address)");
  const char* name = PyUnicode_AsUTF8(args[0]);
  void* at = PyLong_AsVoidPtr(args[1]);
  if (!name || PyErr_Occurred()) return nullptr;
#define SET(NAME)                                                          \
  if (!strcmp(name, #NAME)) {                                              \
    p_##NAME = reinterpret_cast<decltype(&NAME)>(at);                      \
    Py_RETURN_TRUE;                                                        \
  }
  ENTRY_POINTS(SET)
#undef SET
  Py_RETURN_FALSE;
}

#define METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_##NAME)), METH_FASTCALL, nullptr},
PyMethodDef methods[] = {
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bind)), METH_FASTCALL, nullptr},
    ENTRY_POINTS(METHOD){nullptr, nullptr, 0, nullptr}};
#undef METHOD

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mtla_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mtla_call(void) { return PyModule_Create(&module); }
