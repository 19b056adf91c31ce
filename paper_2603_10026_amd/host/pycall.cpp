// CPython entry points for binding.py: turns torch tensors into rf_tensor descriptors and calls
// the C ABI.
//
// Describing a tensor from Python (shape, strides, data pointer, packing) takes about a
// microsecond, a call has up to six of them, and most kernels of a decode step or a small batch
// run for 3 to 10 us: the host was what bounded them.  Here a tensor is read through its C++
// object.  Only plain tensors and parameters are: subclasses, ill-typed arguments and everything
// else that has behaviour of its own in Python go through binding.tensor_desc / binding._stream,
// which also raise the errors.
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "../../include/rf.h"

namespace {

PyObject* g_tensor_desc = nullptr;  // binding.tensor_desc: tensor -> object with rf_tensor's bytes
PyObject* g_stream = nullptr;       // binding._stream: any stream argument -> object with .value

// Fills *d; false with a Python error set on failure.  *on_gpu becomes true for a GPU tensor.
bool describe(PyObject* obj, rf_tensor* d, bool* on_gpu) {
  if (THPVariable_CheckExact(obj)) {
    const at::Tensor& t = THPVariable_Unpack(obj);
    int dtype = -1;
    switch (t.scalar_type()) {
      case at::kFloat: dtype = RF_F32; break;
      case at::kBFloat16: dtype = RF_BF16; break;
      case at::kInt: dtype = RF_I32; break;
      case at::kFloat8_e4m3fn: dtype = RF_FP8_E4M3; break;
      default: break;
    }
    const int64_t n = t.dim();
    if (dtype >= 0 && n >= 1 && n <= RF_MAX_DIMS) {
      std::memset(d, 0, sizeof(*d));
      const auto sizes = t.sizes();
      const auto strides = t.strides();
      bool empty = false;
      for (int64_t i = 0; i < n; ++i) {
        d->shape[i] = sizes[i];
        d->stride[i] = strides[i];
        empty = empty || sizes[i] == 0;
      }
      d->dtype = static_cast<rf_dtype>(dtype);
      d->ndim = static_cast<int>(n);
      d->data = empty ? nullptr : t.data_ptr();
      if (t.is_cuda()) *on_gpu = true;
      return true;
    }
  }
  PyObject* r = PyObject_CallFunctionObjArgs(g_tensor_desc, obj, nullptr);
  if (r == nullptr) return false;
  Py_buffer view;
  const bool ok = PyObject_GetBuffer(r, &view, PyBUF_SIMPLE) == 0;
  if (ok) {
    if (view.len == static_cast<Py_ssize_t>(sizeof(*d))) std::memcpy(d, view.buf, sizeof(*d));
    else PyErr_SetString(PyExc_RuntimeError, "tensor_desc does not have the size of rf_tensor");
    PyBuffer_Release(&view);
  }
  Py_DECREF(r);
  return PyErr_Occurred() == nullptr;
}

bool stream_of(PyObject* obj, bool on_gpu, rf_stream* s) {
  if (obj == Py_None && on_gpu) {  // (a GPU tensor exists, so torch has set up its devices)
    *s = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  PyObject* r = PyObject_CallFunctionObjArgs(g_stream, obj, nullptr);
  PyObject* v = r != nullptr ? PyObject_GetAttrString(r, "value") : nullptr;
  Py_XDECREF(r);
  if (v == nullptr) return false;
  *s = v == Py_None ? nullptr : PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return PyErr_Occurred() == nullptr;
}

bool to_int(PyObject* obj, int* out) {  // int(obj), cut to a C int
  PyObject* v = PyNumber_Long(obj);
  if (v == nullptr) return false;
  *out = static_cast<int>(PyLong_AsUnsignedLongMask(v));
  Py_DECREF(v);
  return PyErr_Occurred() == nullptr;
}

bool to_float(PyObject* obj, float* out) {  // float(obj)
  PyObject* v = PyNumber_Float(obj);
  if (v == nullptr) return false;
  *out = static_cast<float>(PyFloat_AS_DOUBLE(v));
  Py_DECREF(v);
  return true;
}

bool count(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
  return false;
}

// N tensors (from args[0] on), then the stream (last argument).
template <int N>
bool describe_all(PyObject* const* args, Py_ssize_t n, rf_tensor (&d)[N], const int (&at)[N], rf_stream* s) {
  bool on_gpu = false;
  for (int i = 0; i < N; ++i)
    if (!describe(args[at[i]], &d[i], &on_gpu)) return false;
  return stream_of(args[n - 1], on_gpu, s);
}

// The interpreter is free while the C ABI validates and launches.
template <typename F>
PyObject* call(F&& f) {
  rf_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(static_cast<long>(st));
}

PyObject* py_init(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!count(n, 2)) return nullptr;
  Py_INCREF(args[0]);
  Py_INCREF(args[1]);
  Py_XSETREF(g_tensor_desc, args[0]);
  Py_XSETREF(g_stream, args[1]);
  Py_RETURN_NONE;
}

// safe_softmax(x, y, axis, stream)
PyObject* py_safe_softmax(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[2];
  int axis;
  rf_stream s;
  if (!count(n, 4) || !describe_all<2>(args, n, d, {0, 1}, &s) || !to_int(args[2], &axis)) return nullptr;
  return call([&] { return rf_safe_softmax(&d[0], &d[1], axis, s); });
  END_HANDLE_TH_ERRORS
}

// cascade_attention(q, k, v, o, scale, causal, stream)
PyObject* py_cascade_attention(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[4];
  float scale;
  rf_stream s;
  if (!count(n, 7) || !describe_all<4>(args, n, d, {0, 1, 2, 3}, &s) || !to_float(args[4], &scale)) return nullptr;
  const int causal = PyObject_IsTrue(args[5]);
  if (causal < 0) return nullptr;
  return call([&] { return rf_cascade_attention(&d[0], &d[1], &d[2], &d[3], scale, causal, s); });
  END_HANDLE_TH_ERRORS
}

// cascade_attention_splitk(q, k, v, num_splits, part_m, part_l, part_acc, scale, causal, stream)
PyObject* py_cascade_attention_splitk(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[6];
  int splits;
  float scale;
  rf_stream s;
  if (!count(n, 10) || !describe_all<6>(args, n, d, {0, 1, 2, 4, 5, 6}, &s) || !to_int(args[3], &splits) ||
      !to_float(args[7], &scale))
    return nullptr;
  const int causal = PyObject_IsTrue(args[8]);
  if (causal < 0) return nullptr;
  return call([&] {
    return rf_cascade_attention_splitk(&d[0], &d[1], &d[2], splits, &d[3], &d[4], &d[5], scale, causal, s);
  });
  END_HANDLE_TH_ERRORS
}

// merge_states(part_m, part_l, part_acc, o, stream)
PyObject* py_merge_states(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[4];
  rf_stream s;
  if (!count(n, 5) || !describe_all<4>(args, n, d, {0, 1, 2, 3}, &s)) return nullptr;
  return call([&] { return rf_merge_states(&d[0], &d[1], &d[2], &d[3], s); });
  END_HANDLE_TH_ERRORS
}

// rmsnorm_gemm(x, g, w, y, eps, stream)
PyObject* py_rmsnorm_gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[4];
  float eps;
  rf_stream s;
  if (!count(n, 6) || !describe_all<4>(args, n, d, {0, 1, 2, 3}, &s) || !to_float(args[4], &eps)) return nullptr;
  return call([&] { return rf_rmsnorm_gemm(&d[0], &d[1], &d[2], &d[3], eps, s); });
  END_HANDLE_TH_ERRORS
}

// variance(x, mean, var, stream)
PyObject* py_variance(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[3];
  rf_stream s;
  if (!count(n, 4) || !describe_all<3>(args, n, d, {0, 1, 2}, &s)) return nullptr;
  return call([&] { return rf_variance(&d[0], &d[1], &d[2], s); });
  END_HANDLE_TH_ERRORS
}

// fp8_quant_gemm(a, w, c, stream)
PyObject* py_fp8_quant_gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[3];
  rf_stream s;
  if (!count(n, 4) || !describe_all<3>(args, n, d, {0, 1, 2}, &s)) return nullptr;
  return call([&] { return rf_fp8_quant_gemm(&d[0], &d[1], &d[2], s); });
  END_HANDLE_TH_ERRORS
}

// moe_routing(x, w, topk, prob, idx, workspace, stream); workspace: any tensor
PyObject* py_moe_routing(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[4];
  int topk;
  rf_stream s;
  if (!count(n, 7) || !describe_all<4>(args, n, d, {0, 1, 3, 4}, &s) || !to_int(args[2], &topk)) return nullptr;
  void* ws;
  size_t bytes;
  if (THPVariable_CheckExact(args[5])) {
    const at::Tensor& t = THPVariable_Unpack(args[5]);
    ws = t.data_ptr();
    bytes = static_cast<size_t>(t.numel()) * t.element_size();
  } else {
    PyObject* r = PyObject_CallMethod(args[5], "data_ptr", nullptr);
    if (r == nullptr) return nullptr;
    ws = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    PyObject* a = PyObject_CallMethod(args[5], "numel", nullptr);
    PyObject* b = a != nullptr ? PyObject_CallMethod(args[5], "element_size", nullptr) : nullptr;
    PyObject* p = b != nullptr ? PyNumber_Multiply(a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    if (p == nullptr) return nullptr;
    bytes = PyLong_AsSize_t(p);
    Py_DECREF(p);
    if (PyErr_Occurred()) return nullptr;
  }
  return call([&] { return rf_moe_routing(&d[0], &d[1], topk, &d[2], &d[3], ws, bytes, s); });
  END_HANDLE_TH_ERRORS
}

// moe_routing_noalloc(x, w, topk, prob, idx, stream)
PyObject* py_moe_routing_noalloc(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d[4];
  int topk;
  rf_stream s;
  if (!count(n, 6) || !describe_all<4>(args, n, d, {0, 1, 3, 4}, &s) || !to_int(args[2], &topk)) return nullptr;
  return call([&] { return rf_moe_routing_noalloc(&d[0], &d[1], topk, &d[2], &d[3], s); });
  END_HANDLE_TH_ERRORS
}

// describe(tensor) -> the bytes of its rf_tensor
PyObject* py_describe(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  rf_tensor d;
  bool on_gpu = false;
  if (!count(n, 1) || !describe(args[0], &d, &on_gpu)) return nullptr;
  return PyBytes_FromStringAndSize(reinterpret_cast<const char*>(&d), sizeof(d));
  END_HANDLE_TH_ERRORS
}

#define RF_PY(NAME) \
  {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    RF_PY(init), RF_PY(describe), RF_PY(safe_softmax), RF_PY(cascade_attention), RF_PY(cascade_attention_splitk),
    RF_PY(merge_states), RF_PY(rmsnorm_gemm), RF_PY(variance), RF_PY(fp8_quant_gemm), RF_PY(moe_routing),
    RF_PY(moe_routing_noalloc), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rfcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__rfcall() { return PyModule_Create(&module); }
