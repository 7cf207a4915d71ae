// The launch entry points of include/fs.h as CPython calls: addresses taken from the tensors and the call made
// without ctypes in between.  A module of its own, so that the library itself stays free of Python.
//
// A small group is bound by the calls, not by its kernel: with two array objects and a ctypes call around a launch of
// 2.4 us and a kernel of 2.4 us, LayerNorm 256 x 768 fp32 took 4.9 us a call, now 4.2; calls of one microsecond's
// kernels 5.0 -> 3.85.  What is left is HIP's launch (a bare loop of launches in C++ runs at 2.2 to 2.5 us each).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <new>

#include "../../include/fs.h"

namespace {

using LaunchFn = fs_status (*)(fs_plan*, const void* const*, int32_t, void* const*, int32_t, void*);

LaunchFn g_launch = nullptr, g_launch_static = nullptr;     // of the library that the binding has loaded, set once by bind()
PyObject* g_source = nullptr;                               // gives the next two, asked once
PyObject* g_raw_stream = nullptr;                           // device ordinal -> handle of torch's current stream there
PyObject* g_device = nullptr;                               // -> torch's current device; None: the one above takes no ordinal
PyObject* g_c_void_p = nullptr;                             // ctypes.c_void_p
PyObject* g_address_of = nullptr;                           // anything that ctypes takes for a c_void_p -> its address, or None
PyObject* g_data_ptr = nullptr;                             // "data_ptr"

// What ctypes makes of a c_void_p argument: None is NULL, an int is the address, a c_void_p its value; whatever else it
// takes (an object with _as_parameter_ such as a torch stream, an array, a reference) or refuses, ctypes itself is asked.
bool as_handle(PyObject* o, void** out) {
  if (o == Py_None) { *out = nullptr; return true; }
  if (PyLong_Check(o)) {
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
    *out = reinterpret_cast<void*>(static_cast<uintptr_t>(v));
    return true;
  }
  if (!g_address_of) { PyErr_SetString(PyExc_RuntimeError, "bind() has not been called"); return false; }
  PyObject* value = (PyObject*)Py_TYPE(o) == g_c_void_p ? PyObject_GetAttrString(o, "value") : PyObject_CallOneArg(g_address_of, o);
  if (!value) return false;
  bool ok = false;
  if (value == Py_None || PyLong_Check(value)) ok = as_handle(value, out);
  else PyErr_SetString(PyExc_TypeError, "an address is an int or None");
  Py_DECREF(value);
  return ok;
}

bool as_address(PyObject* o, void** out) {
  const unsigned long long v = PyLong_AsUnsignedLongLong(o);
  if (v == (unsigned long long)-1 && PyErr_Occurred()) return false;
  *out = reinterpret_cast<void*>(static_cast<uintptr_t>(v));
  return true;
}

// The device addresses of a list of tensors (anything with data_ptr()) or ints, in a local array or, for long
// lists, one of its own.
struct Addresses {
  void* local[32];
  void** p = local;
  int32_t n = 0;
  ~Addresses() { if (p != local) delete[] p; }

  bool take(PyObject* seq) {
    PyObject* fast;
    if (PyList_Check(seq) || PyTuple_Check(seq)) { fast = seq; Py_INCREF(fast); }
    else {
      if (PyObject_Size(seq) < 0) return false;             // an iterator has no length: refused
      fast = PySequence_List(seq);
      if (!fast) return false;
    }
    const bool ok = read(fast);
    Py_DECREF(fast);
    return ok;
  }

 private:
  bool read(PyObject* fast) {
    const Py_ssize_t count = PySequence_Fast_GET_SIZE(fast);
    if (count > INT32_MAX) { PyErr_SetString(PyExc_OverflowError, "too many tensors"); return false; }
    if (count > (Py_ssize_t)(sizeof local / sizeof *local)) {
      p = new (std::nothrow) void*[count];
      if (!p) { p = local; PyErr_NoMemory(); return false; }
    }
    for (Py_ssize_t i = 0; i < count; ++i) {
      // data_ptr() of a class of the caller's may run anything: its list is looked at anew, its entry is held
      if (i >= PySequence_Fast_GET_SIZE(fast)) { PyErr_SetString(PyExc_RuntimeError, "the list of tensors changed while it was read"); return false; }
      PyObject* t = PySequence_Fast_GET_ITEM(fast, i);
      Py_INCREF(t);
      PyObject* address = PyLong_Check(t) ? t : PyObject_CallMethodNoArgs(t, g_data_ptr);
      bool ok = false;
      if (address && !PyLong_Check(address)) {
        PyObject* index = PyNumber_Index(address);
        Py_DECREF(address);
        address = index;
      }
      if (address) ok = as_address(address, &p[i]);
      if (address != t) Py_XDECREF(address);
      Py_DECREF(t);
      if (!ok) return false;
    }
    n = (int32_t)count;
    return true;
  }
};

// torch's current stream; where to ask is found out the first time (a program that names its streams never imports torch).
bool stream_object(PyObject** stream) {
  if (!g_raw_stream) {
    if (!g_source) { PyErr_SetString(PyExc_RuntimeError, "bind() has not been called"); return false; }
    PyObject* pair = PyObject_CallNoArgs(g_source);
    if (!pair) return false;
    PyObject *raw, *device;
    const bool ok = PyArg_ParseTuple(pair, "OO", &raw, &device);
    if (ok && !g_raw_stream) {
      Py_INCREF(raw);
      Py_INCREF(device);
      g_device = device;
      g_raw_stream = raw;
    }
    Py_DECREF(pair);
    if (!ok) return false;
  }
  if (g_device == Py_None) {
    *stream = PyObject_CallNoArgs(g_raw_stream);
  } else {
    PyObject* device = PyObject_CallNoArgs(g_device);
    *stream = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
    Py_XDECREF(device);
  }
  return *stream != nullptr;
}

bool current_stream(void** out) {
  PyObject* stream;
  if (!stream_object(&stream)) return false;
  const bool ok = as_handle(stream, out);
  Py_DECREF(stream);
  return ok;
}

PyObject* call(LaunchFn fn, void* plan, const Addresses& in, const Addresses& out, void* stream) {
  fs_status st;
  Py_BEGIN_ALLOW_THREADS          // a first launch loads code, and a full queue is waited for
  st = fn(static_cast<fs_plan*>(plan), in.p, in.n, out.p, out.n, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// (plan, inputs, outputs, stream) -> status; stream None: torch's current one
PyObject* launch_with(LaunchFn fn, PyObject* const* args, Py_ssize_t n) {
  if (n != 4) { PyErr_SetString(PyExc_TypeError, "launch(plan, inputs, outputs, stream)"); return nullptr; }
  if (!fn) { PyErr_SetString(PyExc_RuntimeError, "bind() has not been called"); return nullptr; }
  void *plan, *stream;
  Addresses in, out;
  if (args[3] == Py_None ? !current_stream(&stream) : !as_handle(args[3], &stream)) return nullptr;
  if (!as_handle(args[0], &plan) || !in.take(args[1]) || !out.take(args[2])) return nullptr;
  return call(fn, plan, in, out, stream);
}

PyObject* launch(PyObject*, PyObject* const* args, Py_ssize_t n) { return launch_with(g_launch, args, n); }
PyObject* launch_static(PyObject*, PyObject* const* args, Py_ssize_t n) { return launch_with(g_launch_static, args, n); }

// (plan, inputs array, n_in, outputs array, n_out, stream) -> status: host arrays at hand, stream None is the default one
PyObject* launch_arrays(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 6) { PyErr_SetString(PyExc_TypeError, "launch_arrays(plan, inputs, n_in, outputs, n_out, stream)"); return nullptr; }
  if (!g_launch) { PyErr_SetString(PyExc_RuntimeError, "bind() has not been called"); return nullptr; }
  void *plan, *in, *out, *stream;
  if (!as_handle(args[0], &plan) || !as_handle(args[1], &in) || !as_handle(args[3], &out) || !as_handle(args[5], &stream)) return nullptr;
  const long n_in = PyLong_AsLong(args[2]), n_out = PyLong_AsLong(args[4]);
  if ((n_in == -1 || n_out == -1) && PyErr_Occurred()) return nullptr;
  fs_status st;
  Py_BEGIN_ALLOW_THREADS
  st = g_launch(static_cast<fs_plan*>(plan), static_cast<const void* const*>(in), (int32_t)n_in, static_cast<void* const*>(out), (int32_t)n_out, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// (address of fs_launch, address of fs_launch_static, function that says where the current stream comes from, c_void_p,
// function that gives the address of what ctypes takes for one)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  void *a, *b;
  if (n != 5) { PyErr_SetString(PyExc_TypeError, "bind(fs_launch, fs_launch_static, stream_source, c_void_p, address_of)"); return nullptr; }
  if (!as_handle(args[0], &a) || !as_handle(args[1], &b)) return nullptr;
  g_launch = reinterpret_cast<LaunchFn>(a);
  g_launch_static = reinterpret_cast<LaunchFn>(b);
  Py_INCREF(args[2]);
  Py_XSETREF(g_source, args[2]);
  Py_INCREF(args[3]);
  Py_XSETREF(g_c_void_p, args[3]);
  Py_INCREF(args[4]);
  Py_XSETREF(g_address_of, args[4]);
  Py_RETURN_NONE;
}

PyObject* current_stream_handle(PyObject*, PyObject*) {
  PyObject* stream;
  return stream_object(&stream) ? stream : nullptr;
}

#define FASTCALL(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {
    {"bind", FASTCALL(bind), "bind(fs_launch, fs_launch_static, stream_source, c_void_p, address_of): the library's entry points"},
    {"current_stream", current_stream_handle, METH_NOARGS, "the handle of torch's current stream"},
    {"launch", FASTCALL(launch), "launch(plan, inputs, outputs, stream) -> fs_status"},
    {"launch_static", FASTCALL(launch_static), "launch_static(plan, inputs, outputs, stream) -> fs_status"},
    {"launch_arrays", FASTCALL(launch_arrays), "launch_arrays(plan, inputs, n_in, outputs, n_out, stream) -> fs_status"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_launch", "fs_launch and fs_launch_static on Python lists", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__launch() {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  return g_data_ptr ? PyModule_Create(&module) : nullptr;
}
