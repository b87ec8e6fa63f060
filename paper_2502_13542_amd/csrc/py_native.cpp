// The library's entry points for Python: torch tensors in, one C ABI call out.
//
// An eager decode step or a stream of windows is a chain of launches of 3 to 15 us each, so what
// the host spends per call decides its pace.  Marshalled by ctypes, with the checks of every
// tensor in Python, a call took 8 to 11 us (a step of three calls 34 us of host time for 29 us of
// kernels); here the prototypes of actqkv.h drive the conversion and the launch itself is what
// is left of a call.
//
// One template converts the arguments of any entry point from its C++ parameter types: the shape
// (a ctypes structure, by its buffer), integers, floats, int32 and fp32 tensors.  Parameters that
// are plain `void*` take their meaning from a string, one letter per such parameter:
//   s  tensor of the shape's storage type        b  tensor of bf16, whatever the shape says
//   h  like s, but pinned host memory will do    w  workspace (a size_t parameter follows: its bytes)
//   p  address (an integer)                      q  stream, None for the current one
// A tensor parameter accepts None (the library decides whether it may be NULL).
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>
#include <dlfcn.h>

#include <cstring>
#include <string>
#include <tuple>

#include "../../include/actqkv.h"

namespace {

PyObject* g_error = nullptr;         // ActQKVError(code, message)

bool raise(int code, const char* message) {
  PyObject* e = PyObject_CallFunction(g_error, "is", code, message);
  if (e != nullptr) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  return false;
}

struct Args {
  PyObject* const* at;
  PyObject* const* end;
  const char* kinds;
  actqkv_shape shape;
  size_t ws_bytes = 0;
  bool ok = true;

  PyObject* next() {
    if (!ok) return nullptr;
    if (at == end) {
      PyErr_SetString(PyExc_TypeError, "too few arguments");
      ok = false;
      return nullptr;
    }
    return *at++;
  }

  void* tensor(c10::ScalarType want, bool any_type, bool host_too) {
    PyObject* o = next();
    ws_bytes = 0;
    if (o == nullptr || o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) {
      PyErr_SetString(PyExc_TypeError, "expected a tensor or None");
      ok = false;
      return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    // (the runtime is asked about every host tensor: an answer kept by address would outlive the tensor)
    if (!t.is_cuda() && !(host_too && t.is_pinned())) {
      ok = raise(ACTQKV_EINVAL, host_too ? "tensor is neither on the GPU nor in pinned host memory" : "tensor is not on the GPU");
    } else if (!t.is_contiguous()) {
      ok = raise(ACTQKV_EINVAL, "tensor is not contiguous");
    } else if (!any_type && t.scalar_type() != want) {
      ok = raise(ACTQKV_EINVAL, (std::string("tensor dtype ") + c10::toString(t.scalar_type()) + ", expected " +
                                 c10::toString(want)).c_str());
    }
    if (!ok) return nullptr;
    ws_bytes = t.nbytes();
    return t.data_ptr();
  }

  c10::ScalarType storage() const { return shape.dtype == ACTQKV_F32 ? c10::kFloat : c10::kBFloat16; }

  void* opaque() {
    switch (*kinds++) {
      case 's': return tensor(storage(), false, false);
      case 'b': return tensor(c10::kBFloat16, false, false);
      case 'h': return tensor(storage(), false, true);
      case 'w': return tensor(c10::kByte, true, false);
      case 'p': {
        PyObject* o = next();
        void* p = o == nullptr || o == Py_None ? nullptr : PyLong_AsVoidPtr(o);
        if (PyErr_Occurred()) ok = false;
        return p;
      }
      default: {                     // 'q'
        PyObject* o = next();
        if (o == nullptr) return nullptr;
        if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
        void* p = h == nullptr ? nullptr : PyLong_AsVoidPtr(h);
        Py_XDECREF(h);
        if (PyErr_Occurred()) ok = false;
        return p;
      }
    }
  }

  long long integer(long long lo, long long hi) {
    PyObject* o = next();
    if (o == nullptr) return 0;
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
      ok = false;
    } else if (v < lo || v > hi) {
      PyErr_SetString(PyExc_OverflowError, "integer argument out of range");
      ok = false;
    }
    return v;
  }
};

template <typename T> struct Take;
template <> struct Take<const actqkv_shape*> {
  static const actqkv_shape* from(Args& a) {
    PyObject* o = a.next();
    Py_buffer view;
    if (o == nullptr) return nullptr;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
      a.ok = false;
      return nullptr;
    }
    if (view.len != Py_ssize_t(sizeof(actqkv_shape))) {
      PyErr_SetString(PyExc_TypeError, "expected a CShape");
      a.ok = false;
    } else {
      memcpy(&a.shape, view.buf, sizeof(actqkv_shape));
    }
    PyBuffer_Release(&view);
    return &a.shape;
  }
};
template <> struct Take<int> {
  static int from(Args& a) { return int(a.integer(INT32_MIN, INT32_MAX)); }
};
template <> struct Take<int64_t> {
  static int64_t from(Args& a) { return a.integer(INT64_MIN, INT64_MAX); }
};
template <> struct Take<size_t> {    // of a workspace: its bytes; otherwise an argument of its own
  static size_t from(Args& a) { return a.kinds[-1] == 'w' ? a.ws_bytes : size_t(a.integer(0, INT64_MAX)); }
};
template <> struct Take<float> {
  static float from(Args& a) {
    PyObject* o = a.next();
    const double v = o == nullptr ? 0. : PyFloat_AsDouble(o);
    if (o != nullptr && v == -1. && PyErr_Occurred()) a.ok = false;
    return float(v);
  }
};
template <> struct Take<float*> {
  static float* from(Args& a) { return static_cast<float*>(a.tensor(c10::kFloat, false, false)); }
};
template <> struct Take<const float*> : Take<float*> {};
template <> struct Take<int32_t*> {
  static int32_t* from(Args& a) { return static_cast<int32_t*>(a.tensor(c10::kInt, false, false)); }
};
template <> struct Take<const int32_t*> : Take<int32_t*> {};
template <> struct Take<void*> {
  static void* from(Args& a) { return a.opaque(); }
};
template <> struct Take<const void*> : Take<void*> {};

const char* (*g_last_error)() = nullptr;

// An entry point: its name, the letters of its void* parameters, and where load() found it.
template <typename Fn> struct Entry;
template <typename... P> struct Entry<int(P...)> {
  int (*fn)(P...) = nullptr;
  PyObject* call(const char* kinds, PyObject* const* args, Py_ssize_t n) const {
    if (fn == nullptr) {
      PyErr_SetString(PyExc_RuntimeError, "the loaded library does not have this entry point");
      return nullptr;
    }
    // (a tensor without memory, of a fake or a sparse kind for instance, throws when it is asked for an
    // address; C++ exceptions end here, as Python ones)
    HANDLE_TH_ERRORS
    Args a;
    a.at = args;
    a.end = args + n;
    a.kinds = kinds;
    const std::tuple<P...> values{Take<P>::from(a)...};    // (in order: a braced list)
    if (a.ok && a.at != a.end) {
      PyErr_SetString(PyExc_TypeError, "too many arguments");
      a.ok = false;
    }
    if (!a.ok) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS                                 // (a launch waits while its queue is full)
    rc = std::apply(fn, values);
    Py_END_ALLOW_THREADS
    if (rc != ACTQKV_OK) {
      raise(rc, g_last_error != nullptr ? g_last_error() : "");
      return nullptr;
    }
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
  }
};

#define ACTQKV_ENTRIES(X)                                        \
  X(append_kv, "sssssq")                                         \
  X(append_kv_probe, "ssssssq")                                  \
  X(decode_retrieve, "ssssssq")                                  \
  X(decode_select_attention, "bbbbwq")                           \
  X(decode_layer, "bbbbbbbwq")                                   \
  X(retrieval_attention, "sssswq")                               \
  X(retrieval_attention_per_head, "sssswq")                      \
  X(retrieval_attention_static, "ssssq")                         \
  X(retrieval_attention_teams, "sssswqq")                        \
  X(retrieval_attention_windows, "sssswq")                       \
  X(cutoff_budgets, "q")                                         \
  X(cutoff_next_step, "q")                                       \
  X(copy_bytes, "ppq")                                           \
  X(build_probe, "swq")                                          \
  X(gather_blocks, "hhssq")                                      \
  X(gather_blocks_cached, "hhssq")                               \
  X(score_blocks, "sq")                                          \
  X(score_blocks_per_head, "sq")                                 \
  X(select, "q")                                                 \
  X(window_step, "ssssswq")                                      \
  X(decode_step, "ssssssswq")

#define ACTQKV_DEFINE(name, kinds)                                                          \
  Entry<decltype(actqkv_##name)> entry_##name;                                              \
  PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t n) {                     \
    return entry_##name.call(kinds, args, n);                                               \
  }
ACTQKV_ENTRIES(ACTQKV_DEFINE)

// load(path, error class): finds the entry points in the library at `path`
PyObject* py_load(PyObject*, PyObject* args) {
  const char* path;
  PyObject* error;
  if (!PyArg_ParseTuple(args, "sO", &path, &error)) return nullptr;
  void* lib = dlopen(path, RTLD_NOW | RTLD_LOCAL);
  if (lib == nullptr) {
    PyErr_SetString(PyExc_OSError, dlerror());
    return nullptr;
  }
#define ACTQKV_FIND(name, kinds) \
  entry_##name.fn = reinterpret_cast<decltype(&actqkv_##name)>(dlsym(lib, "actqkv_" #name));
  ACTQKV_ENTRIES(ACTQKV_FIND)
  g_last_error = reinterpret_cast<const char* (*)()>(dlsym(lib, "actqkv_last_error"));
  Py_INCREF(error);
  Py_XSETREF(g_error, error);
  Py_RETURN_NONE;
}

#define ACTQKV_METHOD(name, kinds) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(py_##name)), METH_FASTCALL, nullptr},
PyMethodDef g_methods[] = {ACTQKV_ENTRIES(ACTQKV_METHOD){"load", py_load, METH_VARARGS, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&g_module); }
