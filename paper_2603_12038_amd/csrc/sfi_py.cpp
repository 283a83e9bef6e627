// CPython side of the hot calls: arguments of the Python functions in binding.py -> one call of libsfi each.
//
// Why it is native: a fast step of a short context takes the GPU 5 to 7 us, and a call through ctypes took the host 7.4 us
// (torch.cuda.current_stream() alone 2.7 us, a data_ptr() and a conversion per argument the rest), so that a decode loop
// was bound by the marshalling and not by the launch (2.4 us in the HIP runtime).
//
// A tensor argument is anything with a data_ptr() method, an address as an int, a ctypes pointer, or None (null); the last argument
// is the stream: None = torch's current stream, an int handle, or an object with a cuda_stream attribute.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "sfi.h"

namespace {

PyObject* g_error = nullptr;        // SfiError(code, where)
PyObject* g_get_device = nullptr;   // torch: index of the current device
PyObject* g_raw_stream = nullptr;   // torch: handle of the current stream of a device index
PyObject* g_data_ptr = nullptr;     // interned attribute names
PyObject* g_cuda_stream = nullptr;
PyObject* g_value = nullptr;

uint64_t to_word(PyObject* o) {  // any integer, wrapped to 64 bits
  if (PyLong_Check(o)) return PyLong_AsUnsignedLongLongMask(o);
  PyObject* i = PyNumber_Index(o);
  if (i == nullptr) return 0;
  const uint64_t v = PyLong_AsUnsignedLongLongMask(i);
  Py_DECREF(i);
  return v;
}

void* to_pointer(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (PyLong_Check(o)) return reinterpret_cast<void*>(to_word(o));
  PyObject* p = PyObject_CallMethodNoArgs(o, g_data_ptr);
  if (p == nullptr && PyErr_ExceptionMatches(PyExc_AttributeError)) {  // a ctypes pointer (a context handle, say)
    PyObject *type, *value, *trace;
    PyErr_Fetch(&type, &value, &trace);
    p = PyObject_GetAttr(o, g_value);
    if (p == nullptr) {  // neither: the error that names data_ptr
      PyErr_Restore(type, value, trace);
      return nullptr;
    }
    Py_XDECREF(type);
    Py_XDECREF(value);
    Py_XDECREF(trace);
    if (p == Py_None) {
      Py_DECREF(p);
      return nullptr;
    }
  }
  if (p == nullptr) return nullptr;
  void* v = reinterpret_cast<void*>(to_word(p));
  Py_DECREF(p);
  return v;
}

void* to_stream(PyObject* o) {
  PyObject* h;
  if (o == Py_None) {
    PyObject* dev = PyObject_CallNoArgs(g_get_device);
    if (dev == nullptr) return nullptr;
    h = PyObject_CallOneArg(g_raw_stream, dev);
    Py_DECREF(dev);
  } else if (PyLong_Check(o)) {
    return reinterpret_cast<void*>(to_word(o));
  } else {
    h = PyObject_GetAttr(o, g_cuda_stream);
  }
  if (h == nullptr) return nullptr;
  void* v = reinterpret_cast<void*>(to_word(h));
  Py_DECREF(h);
  return v;
}

// (an argument behind one that failed is not looked at: no Python code runs with an exception pending)
template <typename T>
T convert(PyObject* o, bool stream) {
  if (PyErr_Occurred() != nullptr) return T{};
  if constexpr (std::is_pointer_v<T>) return reinterpret_cast<T>(stream ? to_stream(o) : to_pointer(o));
  else return static_cast<T>(to_word(o));
}

template <typename... P, size_t... I>
PyObject* call(int (*fn)(P...), const char* where, PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
  constexpr size_t N = sizeof...(P);
  if (fn == nullptr) return PyErr_Format(PyExc_RuntimeError, "%s: bind() has not been called", where);
  if (n != (Py_ssize_t)N) return PyErr_Format(PyExc_TypeError, "%s takes %zu arguments, got %zd", where, N, n);
  std::tuple<P...> a{convert<P>(args[I], I == N - 1)...};  // braces: left to right
  if (PyErr_Occurred()) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(std::get<I>(a)...);
  Py_END_ALLOW_THREADS
  if (rc == SFI_OK) Py_RETURN_NONE;
  PyObject* e = PyObject_CallFunction(g_error, "is", rc, where);
  if (e != nullptr) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  return nullptr;
}
template <typename... P>
PyObject* call(int (*fn)(P...), const char* where, PyObject* const* args, Py_ssize_t n) {
  return call(fn, where, args, n, std::index_sequence_for<P...>{});
}

#define HOT_CALLS(X)                                                                                                     \
  X(sfi_slow_step) X(sfi_slow_attn) X(sfi_slow_select) X(sfi_evidence_add) X(sfi_evidence_add_causal)                     \
  X(sfi_evidence_select) X(sfi_dense_attn) X(sfi_fast_step) X(sfi_fast_step_static) X(sfi_reorg) X(sfi_fast_step_compact) \
  X(sfi_mixed_step) X(sfi_mixed_step_compact) X(sfi_step_begin) X(sfi_mixed_step_desc) X(sfi_trigger) X(sfi_advance)

// The entry points, handed over by bind: this module is not linked to libsfi, so it works on the very library that
// binding.py has loaded, wherever the package lies and whatever other copies of it are in the process.
#define X(name)                      \
  decltype(&name) fn_##name = nullptr; \
  PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t n) { return call(fn_##name, #name, args, n); }
HOT_CALLS(X)
#undef X

// bind(error class, current-device function, raw-stream function, {entry point: address}): called once by binding.py
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *e, *d, *s, *fns;
  if (!PyArg_ParseTuple(args, "OOOO!", &e, &d, &s, &PyDict_Type, &fns)) return nullptr;
#define X(name)                                                                                            \
  {                                                                                                        \
    PyObject* at = PyDict_GetItemString(fns, #name);                                                       \
    const uint64_t v = at != nullptr ? to_word(at) : 0;                                                    \
    if (PyErr_Occurred()) return nullptr;                                                                  \
    if (v == 0) return PyErr_Format(PyExc_KeyError, "no address of %s", #name);                            \
    fn_##name = reinterpret_cast<decltype(fn_##name)>(v);                                                  \
  }
  HOT_CALLS(X)
#undef X
  Py_INCREF(e); Py_INCREF(d); Py_INCREF(s);
  Py_XSETREF(g_error, e);
  Py_XSETREF(g_get_device, d);
  Py_XSETREF(g_raw_stream, s);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
#define X(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr},
    HOT_CALLS(X)
#undef X
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sfi", "hot calls of libsfi", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sfi(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  g_value = PyUnicode_InternFromString("value");
  if (g_data_ptr == nullptr || g_cuda_stream == nullptr || g_value == nullptr) return nullptr;
  return PyModule_Create(&module);
}
