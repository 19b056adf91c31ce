// CPython entry points for binding.py: turns torch tensors into rf_tensor descriptors and calls
// the C ABI.
//
// Describing a tensor from Python (shape, strides, data pointer, packing) takes about a
// microsecond, a call has up to six of them, and most kernels of a decode step or a small batch
// run for 3 to 10 us: the host was what bounded them.  Here a tensor is read through its C++
// object.  Only plain tensors and parameters are: subclasses, ill-typed arguments and everything
// else that has behaviour of its own in Python go through binding.tensor_desc / binding._stream,
// which also raise the errors.
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "../../include/rf.h"

namespace {

PyObject* g_tensor_desc = nullptr;  // binding.tensor_desc: tensor -> object with rf_tensor's bytes
PyObject* g_stream = nullptr;       // binding._stream: any stream argument -> object with .value

// Fills *d; false with a Python error set on failure.  *device becomes the device of a plain GPU tensor.
bool describe(PyObject* obj, rf_tensor* d, int* device) {
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
      if (t.is_cuda()) *device = t.device().index();
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

bool stream_of(PyObject* obj, int device, rf_stream* s) {
  if (obj == Py_None && device >= 0) {  // (a GPU tensor exists, so torch has set up its devices)
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
bool describe_all(PyObject* const* args, Py_ssize_t n, rf_tensor (&d)[N], const int (&at)[N], rf_stream* s,
                  int* device = nullptr) {
  int dev = -1;
  for (int i = 0; i < N; ++i)
    if (!describe(args[at[i]], &d[i], &dev)) return false;
  if (device != nullptr) *device = dev;
  return stream_of(args[n - 1], dev, s);
}

// Device memory for one call, from torch's caching allocator: it is handed out for the call's stream
// and given back at the end of the call, so that whoever gets it next on that stream runs behind the
// call's kernels, and another stream does not get it.  `data` is null where there is none (no plain
// tensor on the current device, no memory left, an allocator that is not torch's own); the call then
// does without.  So does a call in a capture that torch does not know of: replays of such a graph
// would run on memory that has been handed on.  torch's own captures take from the graph's pool.
// So does a call on hipStreamPerThread: the handle is one, the streams are many, and the allocator goes
// by the handle.  The allocator may have to ask the driver for memory, which a capture in global mode on
// any other thread forbids to threads that have not relaxed their own mode.
class Scratch {
 public:
  Scratch(size_t bytes, int device, rf_stream s) {
    if (bytes == 0 || device < 0) return;
    try {
      const hipStream_t stream = static_cast<hipStream_t>(s);
      if (device != c10::hip::current_device() || stream == hipStreamPerThread) return;
      hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
      if (hipStreamIsCapturing(stream, &capture) != hipSuccess) {
        (void)hipGetLastError();
        return;
      }
      c10::hip::HIPStreamCaptureModeGuard relaxed{hipStreamCaptureModeRelaxed};
      if (capture == hipStreamCaptureStatusNone) {
        data_ = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, stream);
      } else if (stream == c10::hip::getCurrentHIPStream().stream()) {
        data_ = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, stream);
        if (!in_graph_pool()) release();
      }
    } catch (...) {
      release();
    }
  }
  ~Scratch() { release(); }
  Scratch(const Scratch&) = delete;
  Scratch& operator=(const Scratch&) = delete;
  void* data() const { return data_; }

 private:
  void release() {
    if (data_ != nullptr) c10::hip::HIPCachingAllocator::raw_delete(data_);
    data_ = nullptr;
  }
  bool in_graph_pool() const {
    const size_t at = reinterpret_cast<size_t>(data_);
    for (const auto& seg : c10::hip::HIPCachingAllocator::snapshot().segments)
      if (at >= static_cast<size_t>(seg.address) && at - static_cast<size_t>(seg.address) < seg.total_size)
        return seg.owner_private_pool_id.first != 0 || seg.owner_private_pool_id.second != 0;
    return false;
  }
  void* data_ = nullptr;
};

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
  int device;
  if (!count(n, 7) || !describe_all<4>(args, n, d, {0, 1, 2, 3}, &s, &device) || !to_float(args[4], &scale)) return nullptr;
  const int causal = PyObject_IsTrue(args[5]);
  if (causal < 0) return nullptr;
  const size_t bytes = rf_cascade_attention_workspace_bytes(&d[0], &d[1], &d[2], causal);
  const Scratch scratch(bytes, device, s);
  if (scratch.data() != nullptr)
    return call([&] { return rf_cascade_attention_ws(&d[0], &d[1], &d[2], &d[3], scale, causal, scratch.data(), bytes, s); });
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
  int device;
  if (!count(n, 6) || !describe_all<4>(args, n, d, {0, 1, 2, 3}, &s, &device) || !to_float(args[4], &eps)) return nullptr;
  const size_t bytes =
      d[0].ndim == 2 && d[2].ndim == 2 ? rf_rmsnorm_gemm_workspace_bytes(d[0].shape[0], d[0].shape[1], d[2].shape[1]) : 0;
  const Scratch scratch(bytes, device, s);
  if (scratch.data() != nullptr)
    return call([&] { return rf_rmsnorm_gemm_ws(&d[0], &d[1], &d[2], &d[3], eps, scratch.data(), bytes, s); });
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
  int device;
  if (!count(n, 4) || !describe_all<3>(args, n, d, {0, 1, 2}, &s, &device)) return nullptr;
  const size_t bytes =
      d[0].ndim == 2 && d[1].ndim == 2 ? rf_fp8_quant_gemm_workspace_bytes(d[0].shape[0], d[0].shape[1], d[1].shape[0]) : 0;
  const Scratch scratch(bytes, device, s);
  if (scratch.data() != nullptr)
    return call([&] { return rf_fp8_quant_gemm_ws(&d[0], &d[1], &d[2], scratch.data(), bytes, s); });
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
  int device = -1;
  if (!count(n, 1) || !describe(args[0], &d, &device)) return nullptr;
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
