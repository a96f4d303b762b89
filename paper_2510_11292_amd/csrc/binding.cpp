// Python binding of the C ABI in include/louiskv.h: one module function per
// ABI call, with the ABI call's parameters in order.
//
// A decode step of one layer passes 25-40 arguments and runs for 13-40 us, so
// how a call is marshalled decides whether the GPU waits for the host: through
// ctypes (an object for every pointer, a conversion for every argument) one
// step took 14 us of host time, and one of boundary-delimited segments, in
// four calls, 51.  Here the parameter types are read off the ABI function and
// each argument is converted in place:
//   pointers   a tensor (must be contiguous) or None (NULL); an array of
//              handles (void* const*) is passed by its address.  Numbers are
//              refused where a tensor belongs: a kernel would read there
//   stream     the last parameter(s): None (the current stream), a
//              torch.cuda.Stream or a handle
//   numbers    int, bool or float
// The status (or size) comes back as an int, text as a str; the GIL is released
// for the call.
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include <stdexcept>
#include <string>
#include <tuple>
#include <type_traits>
#include <utility>

#include "louiskv.h"

namespace {

struct PyError {};   // a Python exception is set

int64_t to_int(PyObject* o) {
  if (PyLong_Check(o)) return (int64_t)PyLong_AsUnsignedLongLongMask(o);
  PyObject* i = PyNumber_Index(o);
  if (!i) throw PyError();
  const int64_t v = (int64_t)PyLong_AsUnsignedLongLongMask(i);
  Py_DECREF(i);
  return v;
}

[[noreturn]] void not_contiguous() {
  PyErr_SetString(PyExc_ValueError, "libLouisKV needs contiguous tensors");
  throw PyError();
}

void* to_pointer(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (THPVariable_Check(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_contiguous()) not_contiguous();
    return t.data_ptr();
  }
  // anything else that behaves like a tensor
  PyObject* c = PyObject_CallMethod(o, "is_contiguous", nullptr);
  if (!c) throw PyError();
  const int ok = PyObject_IsTrue(c);
  Py_DECREF(c);
  if (ok < 0) throw PyError();
  if (!ok) not_contiguous();
  PyObject* p = PyObject_CallMethod(o, "data_ptr", nullptr);
  if (!p) throw PyError();
  const int64_t v = to_int(p);
  Py_DECREF(p);
  return reinterpret_cast<void*>(v);
}

void* to_array(PyObject* o) {
  return o == Py_None ? nullptr : reinterpret_cast<void*>(to_int(o));
}

void* to_stream(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  if (PyLong_Check(o)) return reinterpret_cast<void*>(PyLong_AsUnsignedLongLongMask(o));
  PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
  if (!h) throw PyError();
  const int64_t v = to_int(h);
  Py_DECREF(h);
  return reinterpret_cast<void*>(v);
}

template <class T>
T convert(PyObject* o, bool stream) {
  if constexpr (std::is_same_v<T, void* const*>) {
    return (T)to_array(o);
  } else if constexpr (std::is_pointer_v<T>) {
    return (T)(stream ? to_stream(o) : to_pointer(o));
  } else if constexpr (std::is_floating_point_v<T>) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PyError();
    return (T)v;
  } else {
    return (T)to_int(o);
  }
}

// Runs f with a C++ exception turned into a Python one.
template <class F>
PyObject* guarded(F&& f) {
  try {
    return f();
  } catch (const PyError&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

template <int kStreams, class R, class... A, std::size_t... I>
PyObject* call(R (*fn)(A...), PyObject* const* args, std::index_sequence<I...>) {
  constexpr std::size_t n = sizeof...(A);
  std::tuple<A...> a{convert<A>(args[I], I + kStreams >= n)...};   // braces: converted in order
  R r;
  Py_BEGIN_ALLOW_THREADS
  r = fn(std::get<I>(a)...);
  Py_END_ALLOW_THREADS
  if constexpr (std::is_same_v<R, const char*>) return PyUnicode_FromString(r);
  else if constexpr (std::is_unsigned_v<R>) return PyLong_FromSize_t(r);
  else return PyLong_FromLong(r);
}

template <class R, class... A>
constexpr std::size_t arity(R (*)(A...)) { return sizeof...(A); }
template <class R, class... A>
std::index_sequence_for<A...> indices(R (*)(A...)) { return {}; }

template <auto kFn, int kStreams>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != (Py_ssize_t)arity(kFn)) {
    PyErr_Format(PyExc_TypeError, "takes %zu arguments, got %zd", arity(kFn), n);
    return nullptr;
  }
  return guarded([&] { return call<kStreams>(kFn, args, decltype(indices(kFn)){}); });
}

// (evicted segment, segments evicted, live tokens, ring slot of the oldest), or the status
PyObject* window_info(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 3) {
      PyErr_SetString(PyExc_TypeError, "takes 3 arguments");
      throw PyError();
    }
    int32_t v[4];
    const int st = louiskv_window_info((int32_t)to_int(args[0]), (int32_t)to_int(args[1]), (int32_t)to_int(args[2]),
                                       &v[0], &v[1], &v[2], &v[3]);
    if (st) return PyLong_FromLong(st);
    return Py_BuildValue("(iiii)", v[0], v[1], v[2], v[3]);
  });
}

#define LKV_ENTRY(name, streams) \
  {#name, reinterpret_cast<PyCFunction>(&entry<&louiskv_##name, streams>), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    {"window_info", reinterpret_cast<PyCFunction>(&window_info), METH_FASTCALL, nullptr},
    LKV_ENTRY(abi_version, 0),
    LKV_ENTRY(status_str, 0),
    LKV_ENTRY(last_error, 0),
    LKV_ENTRY(cluster_prefill_workspace_size, 0),
    LKV_ENTRY(cluster_prefill, 1),
    LKV_ENTRY(pack_pool, 1),
    LKV_ENTRY(cluster_prefill_pipelined_workspace_size, 0),
    LKV_ENTRY(cluster_prefill_pipelined, 2),
    LKV_ENTRY(kmeans_assign, 1),
    LKV_ENTRY(kmeans_update, 1),
    LKV_ENTRY(segment_output, 1),
    LKV_ENTRY(boundary_check, 1),
    LKV_ENTRY(retrieve_workspace_size, 0),
    LKV_ENTRY(retrieve, 1),
    LKV_ENTRY(retrieve_rows_workspace_size, 0),
    LKV_ENTRY(retrieve_rows, 1),
    LKV_ENTRY(sparse_decode_attn_workspace_size, 0),
    LKV_ENTRY(sparse_decode_attn, 1),
    LKV_ENTRY(sparse_decode_attn_rows_workspace_size, 0),
    LKV_ENTRY(sparse_decode_attn_rows, 1),
    LKV_ENTRY(decode_step_workspace_size, 0),
    LKV_ENTRY(decode_step, 1),
    LKV_ENTRY(decode_step_cached_workspace_size, 0),
    LKV_ENTRY(decode_step_cached, 1),
    LKV_ENTRY(sparse_decode_attn_rows_noalloc, 1),
    LKV_ENTRY(decode_prologue, 1),
    LKV_ENTRY(segment_state_ints, 0),
    LKV_ENTRY(segment_state_init, 1),
    LKV_ENTRY(segment_output_boundary, 1),
    LKV_ENTRY(retrieve_seg, 1),
    LKV_ENTRY(retrieve_rows_seg, 1),
    LKV_ENTRY(sparse_decode_attn_seg, 1),
    LKV_ENTRY(sparse_decode_attn_rows_seg, 1),
    LKV_ENTRY(retrieve_delta_workspace_size, 0),
    LKV_ENTRY(retrieve_delta, 1),
    LKV_ENTRY(retrieve_cached, 1),
    LKV_ENTRY(fire_every, 1),
    LKV_ENTRY(page_prefill, 1),
    LKV_ENTRY(retrieve_rows_per_head, 1),
    LKV_ENTRY(sparse_decode_attn_rows_per_head, 1),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
