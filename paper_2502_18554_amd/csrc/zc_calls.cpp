// The hot calls of binding.py in native code: arguments from Python objects to the C ABI of libzc.so and back.
//
// What bounds a small call is the host: a compression of a few thousand values runs for 3 to 4 us, and its caller spent 1.3 us on
// marshalling by ctypes and 3 on the launch.  Here the marshalling is 0.5 us (a chunk of 5120 values compressed and decompressed, each waited for, 22.7 us,
// then 20.5; 16 buffers of 5120 values decompressed by one call 8.2, then 6.4; a waited ring round of 262 177 values 16.4, then 15.0).
// Nothing is decided here: whatever is not of a plain form (lists of other kinds or lengths, negative numbers) is answered with NotImplemented, ahead of
// anything that takes time, and binding.py takes the call its own way, 0.1 us later.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>

#include "../../include/zc.h"

namespace {

struct Calls {
  decltype(&zc_compress_ex) compress;
  decltype(&zc_decompress_ex) decompress;
  decltype(&zc_reduce_compressed_op) reduce;
  decltype(&zc_reduce_step_op) step;
  decltype(&zc_decompress_many) many;
} g_calls;
PyObject *g_device, *g_raw_stream;             // torch's own: the current device, and the current stream's handle on a device
PyObject *g_data_ptr, *g_nbytes, *g_numel, *g_cuda_stream;     // names

// Every reader below returns false where the object is not of a plain form (nothing raised), or with an exception set.
bool exact(PyObject* o, uint64_t& v) {
  if (!PyLong_CheckExact(o)) return false;
  v = PyLong_AsUnsignedLongLong(o);
  if (v == ~uint64_t(0) && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

// Other whole numbers too (numpy's, enumerations), which may run code of their own.
bool whole(PyObject* o, uint64_t& v) {
  if (PyLong_CheckExact(o)) return exact(o, v);
  if (!PyIndex_Check(o)) return false;
  PyObject* const i = PyNumber_Index(o);
  if (!i) return false;
  const bool ok = exact(i, v);
  Py_DECREF(i);
  return ok;
}

bool real(PyObject* o, double& v) {
  v = PyFloat_AsDouble(o);
  if (v != -1.0 || !PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

bool small(PyObject* o, int& v) {
  uint64_t u;
  if (!whole(o, u) || u > 0x7fffffff) return false;
  v = int(u);
  return true;
}

bool of_method(PyObject* tensor, PyObject* name, uint64_t& v) {
  PyObject* r = PyObject_CallMethodNoArgs(tensor, name);
  if (!r) return false;
  const bool ok = exact(r, v);
  Py_DECREF(r);
  return ok;
}

bool address(PyObject* tensor, void*& p) {
  uint64_t v = 0;
  if (tensor != Py_None && !of_method(tensor, g_data_ptr, v)) return false;
  p = reinterpret_cast<void*>(v);
  return true;
}

bool of_attribute(PyObject* o, PyObject* name, uint64_t& v) {
  PyObject* r = PyObject_GetAttr(o, name);
  if (!r) return false;
  const bool ok = exact(r, v);
  Py_DECREF(r);
  return ok;
}
bool bytes_of(PyObject* tensor, uint64_t& v) { return of_attribute(tensor, g_nbytes, v); }

// A capacity: as given (read ahead of all else), or the tensor's own (bytes, or elements).
bool given_capacity(PyObject* given, uint64_t& v) { return given == Py_None || whole(given, v); }
bool own_capacity(PyObject* given, PyObject* tensor, bool elements, uint64_t& v) {
  if (given != Py_None) return true;
  if (!elements) return bytes_of(tensor, v);
  v = 0;
  return tensor == Py_None || of_method(tensor, g_numel, v);
}

// The stream as given, or the current one.
bool stream_of(PyObject* given, void*& stream) {
  uint64_t v = 0;
  if (given != Py_None) {
    if (!of_attribute(given, g_cuda_stream, v)) return false;
    stream = reinterpret_cast<void*>(v);
    return true;
  }
  PyObject* device = PyObject_CallNoArgs(g_device);
  if (!device) return false;
  PyObject* r = PyObject_CallOneArg(g_raw_stream, device);
  Py_DECREF(device);
  if (!r) return false;
  const bool ok = exact(r, v);
  Py_DECREF(r);
  stream = reinterpret_cast<void*>(v);
  return ok;
}

PyObject* not_this_way() {
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NOTIMPLEMENTED;
}

PyObject* answer(int st, bool sync, size_t size) {
  PyObject* const t = PyTuple_New(2);
  if (!t) return nullptr;
  PyObject* const status = PyLong_FromLong(st);
  PyObject* const value = sync ? PyLong_FromSize_t(size) : Py_NewRef(Py_None);
  PyTuple_SET_ITEM(t, 0, status);
  PyTuple_SET_ITEM(t, 1, value);
  if (!status || !value) {
    Py_DECREF(t);
    return nullptr;
  }
  return t;
}

// Lists of k entries each.
PyObject** entries(PyObject* list, Py_ssize_t k) {
  if (!(PyList_CheckExact(list) || PyTuple_CheckExact(list)) || PySequence_Fast_GET_SIZE(list) != k) return nullptr;
  return PySequence_Fast_ITEMS(list);
}
bool addresses(PyObject* list, Py_ssize_t k, const void** to) {
  // (an item is held while its method runs; the list is asked for it each time, in case that changes it)
  for (Py_ssize_t i = 0; i < k; ++i) {
    PyObject** const items = entries(list, k);
    if (!items) return false;
    PyObject* const item = Py_NewRef(items[i]);
    uint64_t v = 0;
    const bool ok = of_method(item, g_data_ptr, v);
    Py_DECREF(item);
    if (!ok) return false;
    to[i] = reinterpret_cast<void*>(v);
  }
  return true;
}
bool counts(PyObject* list, Py_ssize_t k, size_t* to) {
  PyObject** const items = entries(list, k);
  if (!items) return false;
  for (Py_ssize_t i = 0; i < k; ++i) {
    uint64_t v;
    if (!exact(items[i], v)) return false;      // (nothing runs that could change the list)
    to[i] = size_t(v);
  }
  return true;
}

// (d_in, n, abs_eb, d_out, d_ws, sync, stream, out_cap, flags)
PyObject* compress(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  void *in, *out, *ws, *stream;
  uint64_t n, cap, ws_bytes;
  int flags;
  double eb64;
  if (n_args != 9 || !whole(a[1], n) || !real(a[2], eb64) || !small(a[8], flags) || !given_capacity(a[7], cap) || !address(a[0], in) || !address(a[3], out) ||
      !own_capacity(a[7], a[3], false, cap) || !address(a[4], ws) || !bytes_of(a[4], ws_bytes) || !stream_of(a[6], stream))
    return not_this_way();
  const int sync = PyObject_IsTrue(a[5]);
  if (sync < 0) return nullptr;
  const float eb = float(eb64);
  size_t size = 0;
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = g_calls.compress(static_cast<const float*>(in), n, eb, out, cap, sync ? &size : nullptr, ws, ws_bytes, stream, unsigned(flags));
  Py_END_ALLOW_THREADS
  return answer(st, sync, size);
}

// (d_in, in_bytes, d_out, d_ws, sync, stream, out_cap_elems, flags)
PyObject* decompress(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  void *in, *out, *ws, *stream;
  uint64_t in_bytes, cap, ws_bytes;
  int flags;
  if (n_args != 8 || !whole(a[1], in_bytes) || !small(a[7], flags) || !given_capacity(a[6], cap) || !address(a[0], in) || !address(a[2], out) ||
      !own_capacity(a[6], a[2], true, cap) || !address(a[3], ws) || !bytes_of(a[3], ws_bytes) || !stream_of(a[5], stream))
    return not_this_way();
  const int sync = PyObject_IsTrue(a[4]);
  if (sync < 0) return nullptr;
  size_t n = 0;
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = g_calls.decompress(in, in_bytes, static_cast<float*>(out), cap, sync ? &n : nullptr, ws, ws_bytes, stream, unsigned(flags));
  Py_END_ALLOW_THREADS
  return answer(st, sync, n);
}

// (d_chunk, chunk_bytes, d_local, n_local, op, d_out, d_ws, sync, stream, out_cap, flags)
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  void *in, *local, *out, *ws, *stream;
  uint64_t in_bytes, n, cap, ws_bytes;
  int op, flags;
  if (n_args != 11 || !whole(a[1], in_bytes) || !whole(a[3], n) || !small(a[4], op) || !small(a[10], flags) || !given_capacity(a[9], cap) ||
      !address(a[0], in) || !address(a[2], local) || !address(a[5], out) || !own_capacity(a[9], a[5], false, cap) || !address(a[6], ws) || !bytes_of(a[6], ws_bytes) ||
      !stream_of(a[8], stream))
    return not_this_way();
  const int sync = PyObject_IsTrue(a[7]);
  if (sync < 0) return nullptr;
  size_t size = 0;
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = g_calls.step(in, in_bytes, static_cast<const float*>(local), n, op, out, cap, sync ? &size : nullptr, ws, ws_bytes, stream, unsigned(flags));
  Py_END_ALLOW_THREADS
  return answer(st, sync, size);
}

// (d_chunks, chunk_bytes, op, d_out, d_ws, sync, stream, out_cap, flags)
PyObject* reduce(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  void *out, *ws, *stream;
  uint64_t cap, ws_bytes;
  int op, flags;
  const void* chunks[ZC_MAX_K];
  size_t sizes[ZC_MAX_K];
  if (n_args != 9 || !(PyList_CheckExact(a[0]) || PyTuple_CheckExact(a[0]))) return not_this_way();
  const Py_ssize_t k = PySequence_Fast_GET_SIZE(a[0]);
  if (k < 1 || k > ZC_MAX_K || !small(a[2], op) || !small(a[8], flags) || !given_capacity(a[7], cap) || !counts(a[1], k, sizes) || !addresses(a[0], k, chunks) ||
      !address(a[3], out) || !own_capacity(a[7], a[3], false, cap) || !address(a[4], ws) || !bytes_of(a[4], ws_bytes) || !stream_of(a[6], stream))
    return not_this_way();
  const int sync = PyObject_IsTrue(a[5]);
  if (sync < 0) return nullptr;
  size_t size = 0;
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = g_calls.reduce(chunks, sizes, int(k), op, out, cap, sync ? &size : nullptr, ws, ws_bytes, stream, unsigned(flags));
  Py_END_ALLOW_THREADS
  return answer(st, sync, size);
}

// (d_chunks, chunk_bytes, d_outs, d_ws, sync, stream, out_cap_elems, flags)
PyObject* many(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  void *ws, *stream;
  uint64_t ws_bytes;
  int flags;
  const void *chunks[ZC_MAX_K], *outs[ZC_MAX_K];
  size_t sizes[ZC_MAX_K], caps[ZC_MAX_K], ns[ZC_MAX_K] = {};
  if (n_args != 8 || !(PyList_CheckExact(a[0]) || PyTuple_CheckExact(a[0]))) return not_this_way();
  const Py_ssize_t k = PySequence_Fast_GET_SIZE(a[0]);
  if (k < 1 || k > ZC_MAX_K || !small(a[7], flags) || !counts(a[1], k, sizes) || (a[6] != Py_None && !counts(a[6], k, caps)) || !addresses(a[0], k, chunks) ||
      !addresses(a[2], k, outs))
    return not_this_way();
  if (a[6] == Py_None) {
    for (Py_ssize_t i = 0; i < k; ++i) {
      PyObject** const items = entries(a[2], k);
      if (!items) return not_this_way();
      PyObject* const item = Py_NewRef(items[i]);
      uint64_t v = 0;
      const bool ok = of_method(item, g_numel, v);
      Py_DECREF(item);
      if (!ok) return not_this_way();
      caps[i] = size_t(v);
    }
  }
  if (!address(a[3], ws) || !bytes_of(a[3], ws_bytes) || !stream_of(a[5], stream)) return not_this_way();
  const int sync = PyObject_IsTrue(a[4]);
  if (sync < 0) return nullptr;
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = g_calls.many(chunks, sizes, int(k), reinterpret_cast<float* const*>(const_cast<void* const*>(reinterpret_cast<const void* const*>(outs))), caps, sync ? ns : nullptr, ws,
                    ws_bytes, stream, unsigned(flags));
  Py_END_ALLOW_THREADS
  if (!sync) return answer(st, false, 0);
  PyObject* const list = PyList_New(k);
  if (!list) return nullptr;
  for (Py_ssize_t i = 0; i < k; ++i) {
    PyObject* const v = PyLong_FromSize_t(ns[i]);
    if (!v) {
      Py_DECREF(list);
      return nullptr;
    }
    PyList_SET_ITEM(list, i, v);
  }
  return Py_BuildValue("(iN)", st, list);
}

// (addresses of the five calls in the order of Calls, torch's current device, its raw current stream)
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  uint64_t at[5];
  if (n_args != 7) {
    PyErr_SetString(PyExc_TypeError, "setup takes seven arguments");
    return nullptr;
  }
  for (int i = 0; i < 5; ++i)
    if (!whole(a[i], at[i]) || !at[i]) {
      PyErr_SetString(PyExc_ValueError, "setup: the address of a call is missing");
      return nullptr;
    }
  g_calls.compress = reinterpret_cast<decltype(g_calls.compress)>(at[0]);
  g_calls.decompress = reinterpret_cast<decltype(g_calls.decompress)>(at[1]);
  g_calls.reduce = reinterpret_cast<decltype(g_calls.reduce)>(at[2]);
  g_calls.step = reinterpret_cast<decltype(g_calls.step)>(at[3]);
  g_calls.many = reinterpret_cast<decltype(g_calls.many)>(at[4]);
  PyObject* const device = g_device;
  PyObject* const raw = g_raw_stream;
  g_device = Py_NewRef(a[5]);
  g_raw_stream = Py_NewRef(a[6]);
  Py_XDECREF(device);
  Py_XDECREF(raw);
  Py_RETURN_NONE;
}

template <typename F>
PyMethodDef method(const char* name, F f) { return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}; }

PyMethodDef g_methods[] = {method("setup", setup), method("compress", compress), method("decompress", decompress), method("step", step),
                           method("reduce", reduce), method("many", many), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_zc_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__zc_calls() {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  g_nbytes = PyUnicode_InternFromString("nbytes");
  g_numel = PyUnicode_InternFromString("numel");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!g_data_ptr || !g_nbytes || !g_numel || !g_cuda_stream) return nullptr;
  return PyModule_Create(&g_module);
}
