// Native argument marshalling of the Python binding (CPython extension
// _moecall): the per-batch entry points of moe.h called with tensors.
//
// Through ctypes a call cost about 9.5 us of host time (some twenty
// conversions, a Stream object, the foreign call), three times what the small
// kernels behind it take on the GPU.  Here the tensors' device addresses are
// read through the C API of the interpreter and the function is called
// directly: a layout + dispatch + combine step of 128 tokens went from 28.6
// to 16 us back to back on MI355X.
//
// Each function takes its Python arguments by position, as moe.py passes
// them, and returns the entry point's code.  A tensor is any object with
// is_cuda, data_ptr(), numel() and element_size(); None is a null pointer.
// The stream argument is None (the current stream) or has cuda_stream.

#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <dlfcn.h>

#include "moe.h"

namespace {

PyObject* s_is_cuda;
PyObject* s_data_ptr;
PyObject* s_numel;
PyObject* s_element_size;
PyObject* s_shape;
PyObject* s_cuda_stream;
PyObject* s_value;
PyObject* g_argument_error;   // ctypes.ArgumentError
PyObject* g_c_int;            // ctypes.c_int
PyObject* g_get_device;       // () -> index of the current device
PyObject* g_get_stream;       // (index) -> address of its current stream

#define MOE_CALLS(X)                                                                     \
  X(moe_layout) X(moe_layout_fixed) X(moe_dispatch) X(moe_combine) X(moe_layout_dedup) \
  X(moe_dispatch_dedup) X(moe_expand) X(moe_combine_local) X(moe_combine_dedup)
#define X(name) decltype(&name) f_##name;
MOE_CALLS(X)
#undef X

// Reads one call's arguments in order; after the first failure (a Python
// exception is set) everything reads as zero.
class Args {
 public:
  Args(PyObject* const* args, Py_ssize_t n) : args_(args), n_(n) {}
  bool ok() const { return ok_; }

  void expect(Py_ssize_t n) {
    if (n_ != n) {
      PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", n, n_);
      ok_ = false;
    }
  }

  // An integer as a ctypes c_int parameter takes it: anything with __index__,
  // or a c_int.
  unsigned long long integer(PyObject* o) {
    if (PyLong_CheckExact(o)) return PyLong_AsUnsignedLongLongMask(o);
    PyObject* v = nullptr;
    if (PyIndex_Check(o))
      v = PyNumber_Index(o);
    else if (PyObject_IsInstance(o, g_c_int) == 1)
      v = PyObject_GetAttr(o, s_value);
    if (!v) {
      PyErr_Clear();
      PyErr_Format(g_argument_error, "TypeError: wrong type %.100s", Py_TYPE(o)->tp_name);
      ok_ = false;
      return 0;
    }
    const unsigned long long r = PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    return r;
  }

  int i32() { return ok_ ? (int)integer(args_[at_++]) : 0; }

  // Truth of an attribute, or a method's integer result.
  long long method(PyObject* o, PyObject* name) {
    if (!ok_) return 0;
    PyObject* r = PyObject_CallMethodNoArgs(o, name);
    if (!r) {
      ok_ = false;
      return 0;
    }
    const long long v = (long long)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    if (PyErr_Occurred()) ok_ = false;
    return v;
  }

  template <typename T>
  T* ptr() {
    if (!ok_) return nullptr;
    PyObject* o = args_[at_++];
    if (o == Py_None) return nullptr;
    PyObject* c = PyObject_GetAttr(o, s_is_cuda);
    const int cuda = c ? PyObject_IsTrue(c) : -1;
    Py_XDECREF(c);
    if (cuda <= 0) {
      if (cuda == 0) PyErr_SetString(PyExc_ValueError, "libmoe takes device tensors only");
      ok_ = false;
      return nullptr;
    }
    return reinterpret_cast<T*>((uintptr_t)method(o, s_data_ptr));
  }

  // topk_idx: address and its two sizes.
  const int32_t* table(int64_t& T, int& k) {
    T = 0;
    k = 0;
    if (!ok_) return nullptr;
    PyObject* shape = PyObject_GetAttr(args_[at_], s_shape);
    PyObject* seq = shape ? PySequence_Fast(shape, "topk_idx.shape is not a sequence") : nullptr;
    Py_XDECREF(shape);
    if (!seq) {
      ok_ = false;
      return nullptr;
    }
    if (PySequence_Fast_GET_SIZE(seq) != 2) {
      PyErr_SetString(PyExc_ValueError, "topk_idx has two dimensions: tokens and slots");
      ok_ = false;
    } else {
      T = (int64_t)integer(PySequence_Fast_GET_ITEM(seq, 0));
      k = (int)integer(PySequence_Fast_GET_ITEM(seq, 1));
    }
    Py_DECREF(seq);
    return ptr<const int32_t>();
  }

  void* workspace(size_t& bytes) {
    PyObject* o = ok_ ? args_[at_] : nullptr;
    void* p = ptr<void>();
    bytes = ok_ ? (size_t)(method(o, s_numel) * method(o, s_element_size)) : 0;
    return p;
  }

  void* stream() {
    if (!ok_) return nullptr;
    PyObject* o = args_[at_++];
    PyObject* v;
    if (o == Py_None) {
      PyObject* dev = PyObject_CallNoArgs(g_get_device);
      v = dev ? PyObject_CallOneArg(g_get_stream, dev) : nullptr;
      Py_XDECREF(dev);
    } else {
      v = PyObject_GetAttr(o, s_cuda_stream);
    }
    if (!v) {
      ok_ = false;
      return nullptr;
    }
    const uintptr_t s = (uintptr_t)integer(v);
    Py_DECREF(v);
    return reinterpret_cast<void*>(s);
  }

 private:
  PyObject* const* args_;
  Py_ssize_t n_;
  Py_ssize_t at_ = 0;
  bool ok_ = true;
};

// Calls f without the interpreter lock, as ctypes does.
template <typename F>
PyObject* finish(const Args& a, F&& f) {
  if (!a.ok()) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

template <bool FIXED>
PyObject* layout(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Args a(args, n);
  a.expect(FIXED ? 13 : 12);
  int64_t T;
  int k;
  const int32_t* idx = a.table(T, k);
  const int E = a.i32(), R = a.i32(), C = FIXED ? a.i32() : 0;
  int32_t* ec = a.ptr<int32_t>();
  int32_t* eo = a.ptr<int32_t>();
  int32_t* rc = a.ptr<int32_t>();
  int32_t* ro = a.ptr<int32_t>();
  int32_t* pos = a.ptr<int32_t>();
  int32_t* src = a.ptr<int32_t>();
  size_t bytes;
  void* ws = a.workspace(bytes);
  uint32_t* status = a.ptr<uint32_t>();
  void* stream = a.stream();
  return finish(a, [&] {
    return FIXED ? f_moe_layout_fixed(idx, T, k, E, R, C, ec, eo, rc, ro, pos, src, ws, bytes,
                                      status, stream)
                 : f_moe_layout(idx, T, k, E, R, ec, eo, rc, ro, pos, src, ws, bytes, status,
                                stream);
  });
}

// moe_dispatch and, over pair rows, moe_dispatch_dedup: the same arguments.
template <bool DEDUP>
PyObject* dispatch(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Args a(args, n);
  a.expect(16);
  const void* x = a.ptr<const void>();
  const float* xs = a.ptr<const float>();
  const int dtype = a.i32(), H = a.i32(), E = a.i32(), R = a.i32();
  int64_t T;
  int k;
  const int32_t* idx = a.table(T, k);
  const int32_t* pos = a.ptr<const int32_t>();
  const int32_t* ro = a.ptr<const int32_t>();
  const uint64_t* rx = a.ptr<const uint64_t>();
  const uint64_t* rs = a.ptr<const uint64_t>();
  const int32_t* cap = a.ptr<const int32_t>();
  size_t bytes;
  const void* ws = a.workspace(bytes);
  uint32_t* status = a.ptr<uint32_t>();
  void* stream = a.stream();
  const int pitch = a.i32();
  return finish(a, [&] {
    return (DEDUP ? f_moe_dispatch_dedup : f_moe_dispatch)(x, xs, dtype, T, H, k, E, R, idx, pos,
                                                           ro, rx, rs, pitch, cap, ws, bytes,
                                                           status, stream);
  });
}

PyObject* combine(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Args a(args, n);
  a.expect(13);
  const uint64_t* ey = a.ptr<const uint64_t>();
  const float* w = a.ptr<const float>();
  const int H = a.i32(), E = a.i32(), R = a.i32();
  int64_t T;
  int k;
  const int32_t* idx = a.table(T, k);
  const int32_t* pos = a.ptr<const int32_t>();
  const int32_t* ro = a.ptr<const int32_t>();
  const int32_t* cap = a.ptr<const int32_t>();
  uint16_t* y = a.ptr<uint16_t>();
  size_t bytes;
  const void* ws = a.workspace(bytes);
  uint32_t* status = a.ptr<uint32_t>();
  void* stream = a.stream();
  return finish(a, [&] {
    return f_moe_combine(ey, w, T, H, k, E, R, idx, pos, ro, cap, y, ws, bytes, status, stream);
  });
}

PyObject* layout_dedup(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Args a(args, n);
  a.expect(10);
  int64_t T;
  int k;
  const int32_t* idx = a.table(T, k);
  const int E = a.i32(), R = a.i32();
  int32_t* tc = a.ptr<int32_t>();
  int32_t* to = a.ptr<int32_t>();
  int32_t* tp = a.ptr<int32_t>();
  int32_t* ts = a.ptr<int32_t>();
  size_t bytes;
  void* ws = a.workspace(bytes);
  uint32_t* status = a.ptr<uint32_t>();
  void* stream = a.stream();
  return finish(a, [&] {
    return f_moe_layout_dedup(idx, T, k, E, R, tc, to, tp, ts, ws, bytes, status, stream);
  });
}

PyObject* expand(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Args a(args, n);
  a.expect(19);
  const uint64_t* dx = a.ptr<const uint64_t>();
  const uint64_t* ds = a.ptr<const uint64_t>();
  const int dtype = a.i32(), H = a.i32(), E = a.i32(), R = a.i32();
  int64_t T;
  int k;
  const int32_t* idx = a.table(T, k);
  const int32_t* pos = a.ptr<const int32_t>();
  const int32_t* ro = a.ptr<const int32_t>();
  const int32_t* tp = a.ptr<const int32_t>();
  const int32_t* to = a.ptr<const int32_t>();
  const int32_t* dcap = a.ptr<const int32_t>();
  const uint64_t* rx = a.ptr<const uint64_t>();
  const uint64_t* rs = a.ptr<const uint64_t>();
  const int32_t* cap = a.ptr<const int32_t>();
  size_t bytes;
  const void* ws = a.workspace(bytes);
  uint32_t* status = a.ptr<uint32_t>();
  void* stream = a.stream();
  const int pitch = a.i32();
  return finish(a, [&] {
    return f_moe_expand(dx, ds, dtype, T, H, k, E, R, idx, pos, ro, tp, to, dcap, rx, rs, pitch,
                        cap, ws, bytes, status, stream);
  });
}

PyObject* combine_local(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Args a(args, n);
  a.expect(16);
  const uint64_t* ey = a.ptr<const uint64_t>();
  const float* w = a.ptr<const float>();
  const int H = a.i32(), E = a.i32(), R = a.i32();
  int64_t T;
  int k;
  const int32_t* idx = a.table(T, k);
  const int32_t* pos = a.ptr<const int32_t>();
  const int32_t* ro = a.ptr<const int32_t>();
  const int32_t* cap = a.ptr<const int32_t>();
  const int32_t* tp = a.ptr<const int32_t>();
  const int32_t* to = a.ptr<const int32_t>();
  const int32_t* pcap = a.ptr<const int32_t>();
  const uint64_t* part = a.ptr<const uint64_t>();
  size_t bytes;
  const void* ws = a.workspace(bytes);
  uint32_t* status = a.ptr<uint32_t>();
  void* stream = a.stream();
  return finish(a, [&] {
    return f_moe_combine_local(ey, w, T, H, k, E, R, idx, pos, ro, cap, tp, to, pcap, part, ws,
                               bytes, status, stream);
  });
}

PyObject* combine_dedup(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Args a(args, n);
  a.expect(12);
  const uint64_t* part = a.ptr<const uint64_t>();
  const int H = a.i32(), E = a.i32(), R = a.i32();
  int64_t T;
  int k;
  const int32_t* idx = a.table(T, k);
  const int32_t* tp = a.ptr<const int32_t>();
  const int32_t* to = a.ptr<const int32_t>();
  const int32_t* pcap = a.ptr<const int32_t>();
  uint16_t* y = a.ptr<uint16_t>();
  size_t bytes;
  const void* ws = a.workspace(bytes);
  uint32_t* status = a.ptr<uint32_t>();
  void* stream = a.stream();
  return finish(a, [&] {
    return f_moe_combine_dedup(part, T, H, k, E, R, idx, tp, to, pcap, y, ws, bytes, status,
                               stream);
  });
}

// init(lib_path, argument_error, c_int, get_device, get_stream): binds the
// entry points of the libmoe.so that is already loaded.
PyObject* init(PyObject*, PyObject* args) {
  const char* path;
  PyObject *err, *c_int, *dev, *stream;
  if (!PyArg_ParseTuple(args, "sOOOO", &path, &err, &c_int, &dev, &stream)) return nullptr;
  void* h = dlopen(path, RTLD_NOW | RTLD_NOLOAD);
  if (!h) {
    PyErr_Format(PyExc_RuntimeError, "%s is not loaded", path);
    return nullptr;
  }
#define X(name)                                                     \
  f_##name = reinterpret_cast<decltype(&name)>(dlsym(h, #name));    \
  if (!f_##name) {                                                  \
    PyErr_SetString(PyExc_RuntimeError, "missing entry point " #name); \
    return nullptr;                                                 \
  }
  MOE_CALLS(X)
#undef X
  Py_INCREF(err);
  Py_XSETREF(g_argument_error, err);
  Py_INCREF(c_int);
  Py_XSETREF(g_c_int, c_int);
  Py_INCREF(dev);
  Py_XSETREF(g_get_device, dev);
  Py_INCREF(stream);
  Py_XSETREF(g_get_stream, stream);
  Py_RETURN_NONE;
}

#define FAST(name, f) {name, reinterpret_cast<PyCFunction>(f), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
    FAST("layout", layout<false>),
    FAST("layout_fixed", layout<true>),
    FAST("dispatch", dispatch<false>),
    FAST("combine", combine),
    FAST("layout_dedup", layout_dedup),
    FAST("dispatch_dedup", dispatch<true>),
    FAST("expand", expand),
    FAST("combine_local", combine_local),
    FAST("combine_dedup", combine_dedup),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_moecall", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__moecall(void) {
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  s_shape = PyUnicode_InternFromString("shape");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  s_value = PyUnicode_InternFromString("value");
  if (!s_is_cuda || !s_data_ptr || !s_numel || !s_element_size || !s_shape || !s_cuda_stream ||
      !s_value)
    return nullptr;
  return PyModule_Create(&module);
}
