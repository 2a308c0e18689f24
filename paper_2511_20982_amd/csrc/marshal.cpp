// CPython side of the ctypes binding's launching entry points: turns the
// arguments of one call into the C ABI's (device pointers from tensors, host
// pointers from numpy arrays) and makes the call with the GIL released.  The
// library itself is loaded by the binding, which hands over the addresses of
// its functions (bind), so both always speak to the same library.
//
// A call of the small shapes is bounded by this: argument by argument in
// Python it took about 7 us of a call's 9 us of host time.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <tuple>
#include <type_traits>
#include <utility>

#include "dopd_attn.h"

namespace {

PyObject* g_data_ptr = nullptr;      // interned "data_ptr"
PyTypeObject* g_shape = nullptr;     // the binding's class of dopd_attn_shape (set_shape)

// Kinds of arguments, one character each in an entry point's signature:
//   s shape (an instance of the class given to set_shape), d device pointer (an object with data_ptr(),
//   or None), h host pointer (an array that exports its buffer, or None),
//   i int32, z size, p address (the stream)
struct Arg {
  long long value = 0;
  Py_buffer buffer;
  bool held = false;
  ~Arg() {
    if (held) PyBuffer_Release(&buffer);
  }
};

// int(o), modulo 2^64 (the callee's type takes its low bits).
bool integer(PyObject* o, long long* out) {
  PyObject* n = PyLong_Check(o) ? (Py_INCREF(o), o) : PyNumber_Long(o);
  if (!n) return false;
  *out = (long long)PyLong_AsUnsignedLongLongMask(n);
  Py_DECREF(n);
  return !(*out == -1 && PyErr_Occurred());
}

bool host_buffer(PyObject* o, Arg& a) {
  if (PyObject_GetBuffer(o, &a.buffer, PyBUF_SIMPLE) != 0) return false;
  a.held = true;
  a.value = (long long)(uintptr_t)a.buffer.buf;
  return true;
}

bool convert(PyObject* o, char kind, Arg& a) {
  switch (kind) {
    case 's':
      // (other objects export buffers too, of any length)
      if (!g_shape || !PyObject_TypeCheck(o, g_shape)) {
        PyErr_Format(PyExc_TypeError, "shape must be a Shape, not %.200s", Py_TYPE(o)->tp_name);
        return false;
      }
      if (!host_buffer(o, a)) return false;
      if (a.buffer.len < (Py_ssize_t)sizeof(dopd_attn_shape)) {
        PyErr_SetString(PyExc_TypeError, "the Shape is shorter than the library's");
        return false;
      }
      return true;
    case 'h':
      return o == Py_None || host_buffer(o, a);
    case 'd': {
      if (o == Py_None) return true;
      PyObject* p = PyObject_CallMethodNoArgs(o, g_data_ptr);
      if (!p) return false;
      const bool ok = integer(p, &a.value);
      Py_DECREF(p);
      return ok;
    }
    default:
      return integer(o, &a.value);
  }
}

template <class T>
T as(const Arg& a) {
  if constexpr (std::is_pointer_v<T>)
    return reinterpret_cast<T>((uintptr_t)a.value);
  else
    return static_cast<T>(a.value);
}

template <class F>
struct Entry;
template <class... A>
struct Entry<dopd_status(A...)> {
  using Fn = dopd_status (*)(A...);
  static constexpr std::size_t kArgs = sizeof...(A);

  template <std::size_t... I>
  static constexpr bool fits(const char* sig, std::index_sequence<I...>) {
    return ((std::is_pointer_v<A> == (sig[I] != 'i' && sig[I] != 'z')) && ...);
  }
  static constexpr bool fits(const char* sig) { return fits(sig, std::index_sequence_for<A...>{}); }

  template <std::size_t... I>
  static dopd_status invoke(Fn f, const Arg* a, std::index_sequence<I...>) {
    return f(as<A>(a[I])...);
  }

  static PyObject* call(Fn f, const char* name, const char* sig, PyObject* const* args, Py_ssize_t n) {
    if (!f) {
      PyErr_SetString(PyExc_RuntimeError, "the library is not bound");
      return nullptr;
    }
    if (n != (Py_ssize_t)kArgs) {
      PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", name, (Py_ssize_t)kArgs, n);
      return nullptr;
    }
    Arg a[kArgs];
    for (std::size_t i = 0; i < kArgs; ++i)
      if (!convert(args[i], sig[i], a[i])) return nullptr;
    dopd_status st;
    Py_BEGIN_ALLOW_THREADS;
    st = invoke(f, a, std::index_sequence_for<A...>{});
    Py_END_ALLOW_THREADS;
    return PyLong_FromLong(st);
  }
};

// name, signature
#define ENTRIES(X)                                                \
  X(dopd_prefill_attn, "sddddddhidzp")                            \
  X(dopd_prefill_paged_attn, "sdddididhdhiddp")                   \
  X(dopd_prefill_paged_attn_split, "sdddididhdhiidddzp")          \
  X(dopd_prefill_paged_attn_fp8, "sdddddididhdhiidddzp")          \
  X(dopd_kv_write, "sddddididdiip")                               \
  X(dopd_kv_write_fp8, "sddddddididdiip")                         \
  X(dopd_decode_attn, "sdddididhiidddzp")                         \
  X(dopd_decode_attn_fp8, "sdddddididhiidddzp")                   \
  X(dopd_decode_attn_noalloc, "sdddididhiiddp")                   \
  X(dopd_kv_pack_for_handoff, "siddididdhdidp")                   \
  X(dopd_kv_unpack_from_handoff, "siddddhiddidip")                \
  X(dopd_kv_write_pack_for_handoff, "sddddididhiddp")             \
  X(dopd_pd_step, "sdddhiddddddhidddddiiddidzp")                  \
  X(dopd_pd_step_fp8, "sdddhiddddddhidddddddiiddidzp")

#define WRAP(name, sig)                                                                       \
  Entry<decltype(name)>::Fn f_##name = nullptr;                                               \
  static_assert(sizeof(sig) - 1 == Entry<decltype(name)>::kArgs, #name ": one kind per argument"); \
  static_assert(Entry<decltype(name)>::fits(sig), #name ": pointer kinds");                   \
  PyObject* w_##name(PyObject*, PyObject* const* args, Py_ssize_t n) {                        \
    return Entry<decltype(name)>::call(f_##name, #name, sig, args, n);                        \
  }
ENTRIES(WRAP)

// bind(name, address): the library's entry point `name` is at `address`.
PyObject* bind(PyObject*, PyObject* args) {
  const char* name;
  unsigned long long address;
  if (!PyArg_ParseTuple(args, "sK", &name, &address)) return nullptr;
#define BIND(n, sig)                                                              \
  if (std::strcmp(name, #n) == 0) {                                               \
    f_##n = reinterpret_cast<Entry<decltype(n)>::Fn>((uintptr_t)address);         \
    Py_RETURN_NONE;                                                               \
  }
  ENTRIES(BIND)
  PyErr_Format(PyExc_KeyError, "no entry point %s", name);
  return nullptr;
}

// set_shape(class): what a shape argument must be an instance of.
PyObject* set_shape(PyObject*, PyObject* cls) {
  if (!PyType_Check(cls)) {
    PyErr_SetString(PyExc_TypeError, "set_shape takes a class");
    return nullptr;
  }
  Py_INCREF(cls);
  Py_XDECREF(g_shape);
  g_shape = reinterpret_cast<PyTypeObject*>(cls);
  Py_RETURN_NONE;
}

#define METHOD(name, sig) {#name, (PyCFunction)(void (*)(void))w_##name, METH_FASTCALL, sig},
PyMethodDef g_methods[] = {ENTRIES(METHOD){"bind", bind, METH_VARARGS, "bind(name, address)"},
                           {"set_shape", set_shape, METH_O, "set_shape(class)"},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  return g_data_ptr ? PyModule_Create(&g_module) : nullptr;
}
