// The Python binding's common calls in native code: operand checks, output
// and workspace allocation, and the library call, for tensors on the current
// stream of their device.
//
// Each function takes its operands as positional arguments (None where the
// caller gave none) and returns the call's result, a nonzero status as an
// int, or None when it does not take the call: any operand that is not
// exactly what the C-ABI expects, a tensor subclass, a tensor without
// storage.  The caller then runs the same call through the Python checks,
// which raise the error or handle the general case, so nothing is decided
// here but the plain valid call.
//
// What it saves is host time on small layers, whose kernels take a few
// microseconds: the 128-token 1152 -> 1152 linear took 33.7 us a call with
// the checks and allocations in Python (two of them under a stream context)
// for 10 us of kernels, and 13.6 here (9.4 since its quantizer is one launch);
// with a kept output and workspace, in MXFP4, 14.5 -> 8.2.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>

#include "solfp4.h"

namespace {

using at::Tensor;

PyObject* current_raw_stream = nullptr;   // torch._C._cuda_getCurrentRawStream

// Thrown (and caught at the entry) when the native path does not take a call.
struct NotTaken {};

const Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotTaken{};
  return THPVariable_Unpack(o);
}

void need(bool ok) {
  if (!ok) throw NotTaken{};
}

// A contiguous GPU tensor of this type and shape (on `dev`, when given).
void need_tensor(const Tensor& t, at::ScalarType type, at::IntArrayRef shape, const at::Device* dev) {
  need(t.is_cuda() && t.scalar_type() == type && t.layout() == at::kStrided && t.sizes() == shape &&
       t.is_contiguous() && (!dev || t.device() == *dev));
}

void need_matrix(const Tensor& t) { need(t.layout() == at::kStrided && t.dim() == 2); }

Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Device& dev) {
  return at::empty(shape, at::TensorOptions().dtype(type).device(dev));
}

// An operand that the caller gives or leaves to the call, and its Python object.
struct Operand {
  Tensor t;
  PyObject* given = nullptr;   // borrowed
  Operand(PyObject* o, at::ScalarType type, at::IntArrayRef shape, const at::Device& dev) {
    if (o != Py_None) {
      t = tensor(o);
      need_tensor(t, type, shape, &dev);
      given = o;
    }
  }
  void allocate(at::ScalarType type, at::IntArrayRef shape, const at::Device& dev) {
    if (!given) t = make(shape, type, dev);
  }
  PyObject* object() const {
    if (!given) return THPVariable_Wrap(t);
    Py_INCREF(given);
    return given;
  }
};

Tensor workspace_arg(PyObject* o, size_t bytes, const at::Device& dev) {
  if (o == Py_None) return Tensor();
  const Tensor& t = tensor(o);
  need(t.is_cuda() && t.scalar_type() == at::kByte && t.layout() == at::kStrided && t.dim() == 1 &&
       t.is_contiguous() && t.device() == dev && t.numel() >= (int64_t)bytes);
  return t;
}

void* ptr(const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
uint8_t* u8(const Tensor& t) { return static_cast<uint8_t*>(ptr(t)); }
uint16_t* u16(const Tensor& t) { return static_cast<uint16_t*>(ptr(t)); }
float* f32(const Tensor& t) { return static_cast<float*>(ptr(t)); }

// The current stream of `dev`, as the C-ABI takes it.
void* stream_of(const at::Device& dev) {
  PyObject* index = PyLong_FromLong(dev.index());
  PyObject* r = index ? PyObject_CallOneArg(current_raw_stream, index) : nullptr;
  Py_XDECREF(index);
  void* s = r ? PyLong_AsVoidPtr(r) : nullptr;
  Py_XDECREF(r);
  if (PyErr_Occurred()) throw NotTaken{};
  return s;
}

struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

template <typename F>
int call(F&& f) {
  NoGil released;
  return f();
}

template <typename F>
PyObject* entry(Py_ssize_t got, Py_ssize_t want, F&& f) {
  if (got != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return f();
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyObject* failed(int status) { return PyLong_FromLong(status); }

// (x, codes, scales, global_scale, workspace) -> (codes, scales, global_scale)
PyObject* nvfp4_quantize_(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return entry(n, 5, [&]() -> PyObject* {
    const Tensor& x = tensor(a[0]);
    need_matrix(x);
    const int64_t rows = x.size(0), K = x.size(1);
    need(K % 16 == 0);
    need_tensor(x, at::kBFloat16, {rows, K}, nullptr);
    const at::Device dev = x.device();
    Operand codes(a[1], at::kByte, {rows, K / 2}, dev), scales(a[2], at::kByte, {rows, K / 16}, dev);
    Operand gs(a[3], at::kFloat, {1}, dev);
    const size_t bytes = nvfp4_quantize_workspace_bytes(rows, K);
    Tensor ws = workspace_arg(a[4], bytes, dev);
    void* stream = stream_of(dev);
    codes.allocate(at::kByte, {rows, K / 2}, dev);
    scales.allocate(at::kByte, {rows, K / 16}, dev);
    gs.allocate(at::kFloat, {1}, dev);
    if (!ws.defined()) ws = make({(int64_t)std::max<size_t>(bytes, 256)}, at::kByte, dev);
    const int rc = call([&] {
      return nvfp4_quantize(u16(x), rows, K, u8(codes.t), u8(scales.t), f32(gs.t), ptr(ws),
                            (size_t)ws.numel(), stream);
    });
    if (rc) return failed(rc);
    return Py_BuildValue("(NNN)", codes.object(), scales.object(), gs.object());
  });
}

// (x, codes, scales) -> (codes, scales)
PyObject* mxfp4_quantize_(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return entry(n, 3, [&]() -> PyObject* {
    const Tensor& x = tensor(a[0]);
    need_matrix(x);
    const int64_t rows = x.size(0), K = x.size(1);
    need(K % 32 == 0);
    need_tensor(x, at::kBFloat16, {rows, K}, nullptr);
    const at::Device dev = x.device();
    Operand codes(a[1], at::kByte, {rows, K / 2}, dev), scales(a[2], at::kByte, {rows, K / 32}, dev);
    void* stream = stream_of(dev);
    codes.allocate(at::kByte, {rows, K / 2}, dev);
    scales.allocate(at::kByte, {rows, K / 32}, dev);
    const int rc = call([&] { return mxfp4_quantize(u16(x), rows, K, u8(codes.t), u8(scales.t), stream); });
    if (rc) return failed(rc);
    return Py_BuildValue("(NN)", codes.object(), scales.object());
  });
}

// (a_codes, a_scales, a_gs, b_codes, b_scales, b_gs, bias, out, workspace) -> out
PyObject* nvfp4_gemm_(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return entry(n, 9, [&]() -> PyObject* {
    const Tensor &ac = tensor(a[0]), &as = tensor(a[1]), &ag = tensor(a[2]);
    const Tensor &bc = tensor(a[3]), &bs = tensor(a[4]), &bg = tensor(a[5]);
    need_matrix(ac);
    need_matrix(bc);
    const int64_t M = ac.size(0), N = bc.size(0), K = 2 * ac.size(1);
    need(K % 16 == 0);
    need_tensor(ac, at::kByte, {M, K / 2}, nullptr);
    const at::Device dev = ac.device();
    need_tensor(as, at::kByte, {M, K / 16}, &dev);
    need_tensor(ag, at::kFloat, {1}, &dev);
    need_tensor(bc, at::kByte, {N, K / 2}, &dev);
    need_tensor(bs, at::kByte, {N, K / 16}, &dev);
    need_tensor(bg, at::kFloat, {1}, &dev);
    Operand bias(a[6], at::kBFloat16, {N}, dev), out(a[7], at::kBFloat16, {M, N}, dev);
    const size_t bytes = nvfp4_gemm_workspace_bytes(M, N, K);
    Tensor ws = workspace_arg(a[8], bytes, dev);
    void* stream = stream_of(dev);
    out.allocate(at::kBFloat16, {M, N}, dev);
    if (!ws.defined() && bytes) ws = make({(int64_t)bytes}, at::kByte, dev);
    const int rc = call([&] {
      return nvfp4_gemm(u8(ac), u8(as), f32(ag), u8(bc), u8(bs), f32(bg), u16(bias.t), u16(out.t), ptr(ws),
                        ws.defined() ? (size_t)ws.numel() : 0, M, N, K, stream);
    });
    return rc ? failed(rc) : out.object();
  });
}

// (a_codes, a_scales, b_codes, b_scales, bias, out) -> out
PyObject* mxfp4_gemm_(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return entry(n, 6, [&]() -> PyObject* {
    const Tensor &ac = tensor(a[0]), &as = tensor(a[1]), &bc = tensor(a[2]), &bs = tensor(a[3]);
    need_matrix(ac);
    need_matrix(bc);
    const int64_t M = ac.size(0), N = bc.size(0), K = 2 * ac.size(1);
    need(K % 32 == 0);
    need_tensor(ac, at::kByte, {M, K / 2}, nullptr);
    const at::Device dev = ac.device();
    need_tensor(as, at::kByte, {M, K / 32}, &dev);
    need_tensor(bc, at::kByte, {N, K / 2}, &dev);
    need_tensor(bs, at::kByte, {N, K / 32}, &dev);
    Operand bias(a[4], at::kBFloat16, {N}, dev), out(a[5], at::kBFloat16, {M, N}, dev);
    void* stream = stream_of(dev);
    out.allocate(at::kBFloat16, {M, N}, dev);
    const int rc = call([&] {
      return mxfp4_gemm(u8(ac), u8(as), u8(bc), u8(bs), u16(bias.t), u16(out.t), M, N, K, stream);
    });
    return rc ? failed(rc) : out.object();
  });
}

// (x, w_codes, w_scales, w_gs, bias, out, workspace) -> out
PyObject* nvfp4_linear_(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return entry(n, 7, [&]() -> PyObject* {
    const Tensor &x = tensor(a[0]), &wc = tensor(a[1]), &ws_ = tensor(a[2]), &wg = tensor(a[3]);
    need_matrix(x);
    need_matrix(wc);
    const int64_t M = x.size(0), K = x.size(1), N = wc.size(0);
    need(K % 16 == 0);
    need_tensor(x, at::kBFloat16, {M, K}, nullptr);
    const at::Device dev = x.device();
    need_tensor(wc, at::kByte, {N, K / 2}, &dev);
    need_tensor(ws_, at::kByte, {N, K / 16}, &dev);
    need_tensor(wg, at::kFloat, {1}, &dev);
    Operand bias(a[4], at::kBFloat16, {N}, dev), out(a[5], at::kBFloat16, {M, N}, dev);
    const size_t bytes = nvfp4_linear_workspace_bytes(M, N, K);
    Tensor ws = workspace_arg(a[6], bytes, dev);
    void* stream = stream_of(dev);
    out.allocate(at::kBFloat16, {M, N}, dev);
    if (!ws.defined()) ws = make({(int64_t)bytes}, at::kByte, dev);
    const int rc = call([&] {
      return nvfp4_linear(u16(x), u8(wc), u8(ws_), f32(wg), u16(bias.t), u16(out.t), ptr(ws),
                          (size_t)ws.numel(), M, N, K, stream);
    });
    return rc ? failed(rc) : out.object();
  });
}

// (x, w_codes, w_scales, bias, out, workspace) -> out
PyObject* mxfp4_linear_(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return entry(n, 6, [&]() -> PyObject* {
    const Tensor &x = tensor(a[0]), &wc = tensor(a[1]), &ws_ = tensor(a[2]);
    need_matrix(x);
    need_matrix(wc);
    const int64_t M = x.size(0), K = x.size(1), N = wc.size(0);
    need(K % 32 == 0);
    need_tensor(x, at::kBFloat16, {M, K}, nullptr);
    const at::Device dev = x.device();
    need_tensor(wc, at::kByte, {N, K / 2}, &dev);
    need_tensor(ws_, at::kByte, {N, K / 32}, &dev);
    Operand bias(a[3], at::kBFloat16, {N}, dev), out(a[4], at::kBFloat16, {M, N}, dev);
    const size_t bytes = mxfp4_linear_workspace_bytes(M, K);
    Tensor ws = workspace_arg(a[5], bytes, dev);
    void* stream = stream_of(dev);
    out.allocate(at::kBFloat16, {M, N}, dev);
    if (!ws.defined()) ws = make({(int64_t)bytes}, at::kByte, dev);
    const int rc = call([&] {
      return mxfp4_linear(u16(x), u8(wc), u8(ws_), u16(bias.t), u16(out.t), ptr(ws), (size_t)ws.numel(), M,
                          N, K, stream);
    });
    return rc ? failed(rc) : out.object();
  });
}

PyMethodDef methods[] = {
    {"nvfp4_quantize", (PyCFunction)(void*)nvfp4_quantize_, METH_FASTCALL, nullptr},
    {"mxfp4_quantize", (PyCFunction)(void*)mxfp4_quantize_, METH_FASTCALL, nullptr},
    {"nvfp4_gemm", (PyCFunction)(void*)nvfp4_gemm_, METH_FASTCALL, nullptr},
    {"mxfp4_gemm", (PyCFunction)(void*)mxfp4_gemm_, METH_FASTCALL, nullptr},
    {"nvfp4_linear", (PyCFunction)(void*)nvfp4_linear_, METH_FASTCALL, nullptr},
    {"mxfp4_linear", (PyCFunction)(void*)mxfp4_linear_, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", "Native checks, allocation and calls of the binding.",
                      -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() {
  PyObject* c = PyImport_ImportModule("torch._C");
  if (!c) return nullptr;
  current_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
  Py_DECREF(c);
  if (!current_raw_stream) return nullptr;
  return PyModule_Create(&module);
}
