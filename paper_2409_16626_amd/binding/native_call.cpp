// Calls into libhif8.so with Python arguments: the marshalling of hif8.py's launch wrappers for the arguments that programs pass all the time,
// in native code.  A call through ctypes spends about 2 us on it, next to 2.5 us of the runtime's kernel launch; here it is a fifth of that (4 x 4096 bfloat16, scaled and
// encoded, 6.1 -> 4.45 us a call; an encode of 18,000 values 5.7 -> 4.4).
//
// Each function takes the arguments of the C call in its order.  Pointers: None, an int, or a torch.Tensor that lies on the GPU and is contiguous; a byte
// count behind a workspace may be None, the size of that tensor; truth values are whole numbers; the stream is None (torch's current one), an int or an
// object with the handle in `cuda_stream`.  What is of another kind (tensor subclasses, CPU tensors, numbers that do not fit, an active torch function mode
// other than that of a default device, which has no part in these calls, ...) is not looked at here: the function returns NotImplemented without having done anything, and hif8.py goes its own way, with its own errors.
// Success returns None; a status other than HIF8_OK raises through the checker that set_up() was given.  The GIL is released during the call,
// as ctypes does: a launch may wait for the queue.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <dlfcn.h>
#include <torch/csrc/PyInterpreter.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <limits>
#include <tuple>
#include <type_traits>
#include <utility>

#include "hif8.h"

namespace {

PyObject* g_check = nullptr;       // check(status): raises
PyObject* g_device = nullptr;      // () -> index of the current device
PyObject* g_raw_stream = nullptr;  // (device) -> handle of its current stream
PyObject* g_device_mode = nullptr; // type of the function mode that a default device is, or None

struct Seen {
  const at::Tensor* last = nullptr;  // tensor of the workspace argument just before
  bool any = false;                  // a GPU tensor among the arguments: the device is initialised
};

bool take_pointer(PyObject* o, void** p, Seen& seen, bool workspace = false) {
  if (o == Py_None) {
    *p = nullptr;
    return true;
  }
  if (PyLong_CheckExact(o)) {
    *p = PyLong_AsVoidPtr(o);
    if (*p == nullptr && PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    return true;
  }
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous()) return false;
  *p = t.data_ptr();
  if (workspace) seen.last = &t;
  seen.any = true;
  return true;
}

template <typename T>
bool take_integer(PyObject* o, T* v, const Seen& seen) {
  if (std::is_same<T, size_t>::value && o == Py_None && seen.last != nullptr) {
    *v = (T)(seen.last->numel() * seen.last->element_size());
    return true;
  }
  if (!PyLong_CheckExact(o) && !PyBool_Check(o)) return false;
  if (std::is_signed<T>::value) {
    const long long x = PyLong_AsLongLong(o);
    if (x == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    if (x < (long long)std::numeric_limits<T>::min() || x > (long long)std::numeric_limits<T>::max()) return false;
    *v = (T)x;
  } else {
    const unsigned long long x = PyLong_AsUnsignedLongLong(o);
    if (x == (unsigned long long)-1 && PyErr_Occurred()) {
      PyErr_Clear();
      return false;
    }
    if (x > (unsigned long long)std::numeric_limits<T>::max()) return false;
    *v = (T)x;
  }
  return true;
}

bool take_float(PyObject* o, float* v) {
  if (PyFloat_CheckExact(o)) {
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
  }
  if (!PyLong_CheckExact(o)) return false;
  const double x = PyLong_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  *v = (float)x;
  return true;
}

bool take_stream(PyObject* o, void** p, const Seen& seen) {
  if (PyLong_CheckExact(o)) {
    Seen none;
    return take_pointer(o, p, none);
  }
  PyObject* handle = nullptr;
  if (o != Py_None) {
    handle = PyObject_GetAttrString(o, "cuda_stream");
  } else if (seen.any) {
    PyObject* device = PyObject_CallNoArgs(g_device);
    handle = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
    Py_XDECREF(device);
  }
  Seen none;
  const bool ok = handle != nullptr && PyLong_CheckExact(handle) && take_pointer(handle, p, none);
  Py_XDECREF(handle);
  if (!ok) PyErr_Clear();
  return ok;
}

template <typename T>
bool take(PyObject* o, T* v, Seen& seen, bool is_stream) {
  if constexpr (std::is_pointer<T>::value) {
    void* p = nullptr;
    if (!(is_stream ? take_stream(o, &p, seen) : take_pointer(o, &p, seen, std::is_same<T, void*>::value))) return false;
    *v = static_cast<T>(p);
    return true;
  } else if constexpr (std::is_floating_point<T>::value) {
    return take_float(o, v);
  } else {
    const bool ok = take_integer(o, v, seen);
    seen.last = nullptr;
    return ok;
  }
}

template <typename... A, size_t... I>
bool take_all(PyObject* const* args, std::tuple<A...>& values, Seen& seen, std::index_sequence<I...>) {
  return (take(args[I], &std::get<I>(values), seen, I + 1 == sizeof...(A)) && ...);  // the stream comes last in every call
}

// whether a function mode is active that may want to see what is done with the tensors
bool seen_by_a_mode() {
  if (!at::impl::torch_function_mode_enabled()) return false;
  for (int64_t i = 0; i < at::impl::PythonTorchFunctionTLS::stack_len(); ++i) {
    PyObject* mode = at::impl::PythonTorchFunctionTLS::get_stack_at(i)->ptr(getPyInterpreter());
    if (reinterpret_cast<PyObject*>(Py_TYPE(mode)) != g_device_mode) return true;
  }
  return false;
}

template <typename... A>
PyObject* run(hif8_status (*fn)(A...), PyObject* const* args, Py_ssize_t n) {
  std::tuple<A...> values{};
  Seen seen;
  try {
    if (fn == nullptr || n != (Py_ssize_t)sizeof...(A) || seen_by_a_mode() ||
        !take_all(args, values, seen, std::index_sequence_for<A...>{}))
      Py_RETURN_NOTIMPLEMENTED;
  } catch (...) {  // a tensor without storage
    PyErr_Clear();
    Py_RETURN_NOTIMPLEMENTED;
  }
  hif8_status status;
  Py_BEGIN_ALLOW_THREADS
  status = std::apply(fn, values);
  Py_END_ALLOW_THREADS
  if (status == HIF8_OK) Py_RETURN_NONE;
  PyObject* message = PyLong_FromLong((long)status);
  PyObject* r = message ? PyObject_CallOneArg(g_check, message) : nullptr;
  Py_XDECREF(message);
  return r;
}

#define KINDS(X, PRE, POST) X(PRE##f32##POST) X(PRE##bf16##POST) X(PRE##f16##POST)
#define FUNCTIONS(X)                                                                                                                   \
  KINDS(X, hif8_amax_, ) KINDS(X, hif8_encode_, ) KINDS(X, hif8_decode_, ) KINDS(X, hif8_fake_quant_, ) KINDS(X, hif8_encode_, _ds)      \
  KINDS(X, hif8_decode_, _ds) KINDS(X, hif8_fake_quant_, _ds) KINDS(X, hif8_encode_, _sr) KINDS(X, hif8_fake_quant_, _sr)                \
  KINDS(X, hif8_quantize_tensor_, ) KINDS(X, hif8_multi_encode_, _ds) KINDS(X, hif8_scale_sweep_, ) KINDS(X, hif8_amax_axis_, )          \
  KINDS(X, hif8_encode_axis_, ) KINDS(X, hif8_decode_axis_, ) KINDS(X, hif8_quantize_rows_, ) KINDS(X, hif8_gemm_, )                     \
  KINDS(X, hif8_gemm_ws_, ) KINDS(X, hif8_gemm_expanded_, ) X(hif8_gemm_sqerr) X(hif8_gemm_ws_sqerr) X(hif8_gemm_expanded_sqerr)         \
  X(hif8_expand_bf16) X(hif8_expand_bf16_t) X(hif8_scale_from_amax) X(hif8_scale_from_amax_n)

// the library's functions, found in the copy that hif8.py has loaded
#define SLOT(NAME) decltype(&NAME) p_##NAME = nullptr;
FUNCTIONS(SLOT)
#undef SLOT

// set_up(handle of the loaded library, check, device, raw_stream, type of the default device's mode or None)
PyObject* set_up(PyObject*, PyObject* const* args, Py_ssize_t n) {
  void* handle = n == 5 ? PyLong_AsVoidPtr(args[0]) : nullptr;
  if (handle == nullptr) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "set_up(library handle, check, device, raw_stream, device_mode)");
    return nullptr;
  }
  const char* missing = nullptr;
#define FIND(NAME)                                                \
  p_##NAME = reinterpret_cast<decltype(&NAME)>(dlsym(handle, #NAME)); \
  if (p_##NAME == nullptr) missing = #NAME;
  FUNCTIONS(FIND)
#undef FIND
  if (missing != nullptr) {
    PyErr_Format(PyExc_ImportError, "libhif8 has no %s", missing);
    return nullptr;
  }
  PyObject** const to[4] = {&g_check, &g_device, &g_raw_stream, &g_device_mode};
  for (int i = 0; i < 4; ++i) {
    Py_INCREF(args[i + 1]);
    Py_XDECREF(*to[i]);
    *to[i] = args[i + 1];
  }
  Py_RETURN_NONE;
}

#define METHOD(NAME)                                                                                                       \
  {#NAME, (PyCFunction)(void (*)(void))(+[](PyObject*, PyObject* const* args, Py_ssize_t n) { return run(p_##NAME, args, n); }), \
   METH_FASTCALL, nullptr},
PyMethodDef methods[] = {{"set_up", (PyCFunction)(void (*)(void))set_up, METH_FASTCALL, nullptr}, FUNCTIONS(METHOD){nullptr, nullptr, 0, nullptr}};
#undef METHOD

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native_call() { return PyModule_Create(&module); }
