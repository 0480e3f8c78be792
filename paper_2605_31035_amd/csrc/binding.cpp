// Native call path of the Python binding: argument checks, output allocation
// and the library call of the functions that a serving or training loop
// calls per layer, in one C++ call each.  At a few tokens the GPU work of a
// call is 3 to 20 us, and marshalling it in Python (three torch.empty, a
// ctypes call with a dozen converted arguments, the stream lookup) took 13 us
// a call.
//
// Every function returns None for arguments that it does not take as they
// are (other types, shapes, layouts or devices, tensor subclasses, active
// torch function modes) or when the library reports an error; the Python
// function then goes on as it would without this module, with its checks and
// error messages.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mixfp4.h"

namespace {

const c10::DispatchKeySet kWrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                    c10::DispatchKey::FuncTorchGradWrapper,
                                    c10::DispatchKey::Functionalize});

// The tensor of a plain torch.Tensor (or Parameter) on the current device
// with memory of its own; NULL otherwise.
const at::Tensor* plain(PyObject* o, at::ScalarType type, int64_t dim = -1) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.key_set().has_any(kWrapped) ||
      t.layout() != at::kStrided || t.is_neg() || t.is_conj())
    return nullptr;
  if (dim >= 0 && t.dim() != dim) return nullptr;
  if (t.device().index() != c10::hip::current_device()) return nullptr;
  return &t;
}

// As plain, of the given shape and contiguous.
const at::Tensor* matrix(PyObject* o, at::ScalarType type, int64_t rows, int64_t cols) {
  const at::Tensor* t = plain(o, type, 2);
  return t && t->size(0) == rows && t->size(1) == cols && t->is_contiguous() ? t : nullptr;
}

// None, or a contiguous fp32 tensor of one element; false when neither.
bool scale_arg(PyObject* o, float** p) {
  *p = nullptr;
  if (o == Py_None) return true;
  const at::Tensor* t = plain(o, at::kFloat);
  if (!t || t->numel() != 1 || !t->is_contiguous()) return false;
  *p = static_cast<float*>(t->data_ptr());
  return true;
}

// Lets other Python threads run, as a ctypes call does, while outputs are
// allocated and the library is called: a launch may wait for room in the
// queue, and a host function in front of it on the stream may need the
// interpreter.  No Python object and no argument's tensor is touched
// meanwhile (another thread may change it): shapes and addresses are read
// before, and the caller's arguments keep the memory alive.
class WithoutGil {
 public:
  WithoutGil() : state_(PyEval_SaveThread()) {}
  ~WithoutGil() { PyEval_RestoreThread(state_); }
  WithoutGil(const WithoutGil&) = delete;
  WithoutGil& operator=(const WithoutGil&) = delete;

 private:
  PyThreadState* state_;
};

bool modes_active() {
  return at::impl::torch_function_mode_enabled() ||
         c10::impl::TorchDispatchModeTLS::any_modes_set();
}

at::Tensor empty(at::IntArrayRef shape, at::ScalarType type, c10::Device device) {
  return at::empty(shape, at::TensorOptions().dtype(type).device(device));
}

uint8_t* bytes(const at::Tensor& t) { return static_cast<uint8_t*>(t.data_ptr()); }
float* floats(const at::Tensor& t) { return static_cast<float*>(t.data_ptr()); }

void* stream_of(c10::Device device) {
  return c10::hip::getCurrentHIPStream(device.index()).stream();
}

PyObject* triple(const at::Tensor& a, const at::Tensor& b, PyObject* c) {
  PyObject* x = THPVariable_Wrap(a);
  PyObject* y = THPVariable_Wrap(b);
  PyObject* r = PyTuple_Pack(3, x, y, c);
  Py_DECREF(x);
  Py_DECREF(y);
  return r;
}

PyObject* triple(const at::Tensor& a, const at::Tensor& b, const at::Tensor& c) {
  PyObject* z = THPVariable_Wrap(c);
  PyObject* r = triple(a, b, z);
  Py_DECREF(z);
  return r;
}

// A quantized operand (codes [rows, k/2], scales [rows, k/16], s32 or None).
struct Operand {
  uint8_t* codes = nullptr;
  uint8_t* scales = nullptr;
  float* s32 = nullptr;
  int64_t rows = 0, k = 0;
  c10::Device device = c10::Device(c10::kCPU);
};
bool operand(PyObject* o, Operand& q) {
  if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 3) return false;
  const at::Tensor* codes = plain(PyTuple_GET_ITEM(o, 0), at::kByte, 2);
  if (!codes || !codes->is_contiguous()) return false;
  q.rows = codes->size(0);
  q.k = 2 * codes->size(1);
  if (q.k % 16 != 0) return false;
  const at::Tensor* scales = matrix(PyTuple_GET_ITEM(o, 1), at::kByte, q.rows, q.k / 16);
  if (!scales) return false;
  q.codes = bytes(*codes);
  q.scales = bytes(*scales);
  q.device = codes->device();
  return scale_arg(PyTuple_GET_ITEM(o, 2), &q.s32);
}

template <typename Body>
PyObject* guarded(Body body) {
  try {
    if (!modes_active()) {
      PyObject* r = body();
      if (r) return r;
      if (PyErr_Occurred()) return nullptr;
    }
  } catch (const std::exception& e) {
    // an allocation that failed: the Python path does without scratch or
    // workspace, or raises as torch does
  }
  Py_RETURN_NONE;
}

// Largest tensor whose rotated copy (2 bytes an element) is taken as scratch:
// 128 MB, so that the extra memory of a call stays bounded (the copy pays for
// any size).
constexpr int64_t kRotatedElems = int64_t(1) << 26;

// quantize(x, tensor_scale, flags, hadamard_block, signs, seed, offset)
PyObject* quantize(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 7) Py_RETURN_NONE;
  return guarded([&]() -> PyObject* {
    const at::Tensor* x = plain(args[0], at::kBFloat16, 2);
    if (!x || x->stride(1) != 1) return nullptr;
    const int64_t rows = x->size(0), k = x->size(1);
    const unsigned flags = (unsigned)PyLong_AsUnsignedLongMask(args[2]);
    const long block = PyLong_AsLong(args[3]);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      return nullptr;
    }
    if (rows <= 0 || k <= 0 || k % 16 != 0 || block < 0 || block > 256) return nullptr;
    float* given;
    if (!scale_arg(args[1], &given)) return nullptr;
    const int8_t* signs = nullptr;
    if (args[4] != Py_None && block == 0) return nullptr;
    if (args[4] != Py_None) {
      const at::Tensor* s = plain(args[4], at::kChar);
      if (!s || !s->is_contiguous() || s->numel() != block) return nullptr;
      signs = static_cast<const int8_t*>(s->data_ptr());
    }
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(args[5]);
    const uint64_t offset = PyLong_AsUnsignedLongLongMask(args[6]);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      return nullptr;
    }
    const bool t = (flags & MIXFP4_TRANSPOSE) != 0;
    const int64_t orows = t ? k : rows, ok = t ? rows : k;
    if (ok % 16 != 0) return nullptr;
    const int64_t room = block >= 128 && !t && rows * k <= kRotatedElems ? 2 * rows * k : 0;
    const uint16_t* xp = static_cast<const uint16_t*>(x->data_ptr());
    const int64_t ldx = x->stride(0);
    const c10::Device dev = x->device();
    at::Tensor codes, scales, ts, scratch;
    int st;
    {
      const WithoutGil released;
      codes = empty({orows, ok / 2}, at::kByte, dev);
      scales = empty({orows, ok / 16}, at::kByte, dev);
      if (!given) ts = empty({1}, at::kFloat, dev);
      if (!given && rows * k > (int64_t(1) << 17))
        scratch = empty({mixfp4_quantize_scratch_bytes() + room}, at::kByte, dev);
      st = mixfp4_quantize_ws(xp, rows, k, ldx, bytes(codes), bytes(scales),
                              given ? given : floats(ts), flags, (int32_t)block, signs, seed,
                              offset, scratch.defined() ? scratch.data_ptr() : nullptr,
                              scratch.defined() ? scratch.numel() : 0, stream_of(dev));
    }
    if (st != MIXFP4_OK) return nullptr;
    return given ? triple(codes, scales, args[1]) : triple(codes, scales, ts);
  });
}

// gemm(a, w, auto)
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) Py_RETURN_NONE;
  return guarded([&]() -> PyObject* {
    Operand a, w;
    if (!operand(args[0], a) || !operand(args[1], w) || a.k != w.k || a.rows <= 0 || w.rows <= 0)
      return nullptr;
    int64_t need = 0;
    const bool automatic = args[2] == Py_True;
    if (automatic && (reinterpret_cast<uintptr_t>(w.scales) & 3u) != 0)
      return nullptr;                    // rare: the Python path sizes its workspace
    if (automatic &&
        mixfp4_gemm_auto_workspace_size(a.rows, w.rows, a.k, &need) != MIXFP4_OK)
      return nullptr;
    at::Tensor c, ws;
    int st;
    {
      const WithoutGil released;
      c = empty({a.rows, w.rows}, at::kFloat, a.device);
      if (need > 0) ws = empty({need}, at::kByte, a.device);
      st = mixfp4_gemm_auto(a.codes, a.scales, a.s32, w.codes, w.scales, w.s32, a.rows, w.rows,
                            a.k, floats(c), need > 0 ? ws.data_ptr() : nullptr, need,
                            stream_of(a.device));
    }
    return st == MIXFP4_OK ? THPVariable_Wrap(c) : nullptr;
  });
}

// decode_step(x, w, sync)
PyObject* decode_step(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) Py_RETURN_NONE;
  return guarded([&]() -> PyObject* {
    const at::Tensor* x = plain(args[0], at::kBFloat16, 2);
    Operand w;
    if (!x || !x->is_contiguous() || !operand(args[1], w)) return nullptr;
    const int64_t m = x->size(0), k = x->size(1);
    if (w.k != k || w.rows <= 0 || m < 1 || m > 16 || k <= 0 || k % 64 != 0) return nullptr;
    const at::Tensor* sync = plain(args[2], at::kInt);
    if (!sync || sync->numel() != 4 || !sync->is_contiguous()) return nullptr;
    const uint16_t* xp = static_cast<const uint16_t*>(x->data_ptr());
    uint32_t* sp = static_cast<uint32_t*>(sync->data_ptr());
    at::Tensor codes, scales, ts, c;
    int st;
    {
      const WithoutGil released;
      codes = empty({m, k / 2}, at::kByte, w.device);
      scales = empty({m, k / 16}, at::kByte, w.device);
      ts = empty({1}, at::kFloat, w.device);
      c = empty({m, w.rows}, at::kFloat, w.device);
      st = mixfp4_decode_step(xp, m, k, w.codes, w.scales, w.s32, w.rows, bytes(codes),
                              bytes(scales), floats(ts), floats(c), sp, stream_of(w.device));
    }
    if (st != MIXFP4_OK) return nullptr;
    PyObject* q = triple(codes, scales, ts);
    PyObject* o = THPVariable_Wrap(c);
    PyObject* r = PyTuple_Pack(2, o, q);
    Py_DECREF(o);
    Py_DECREF(q);
    return r;
  });
}

// dequantize(codes, scales, tensor_scale)
PyObject* dequantize(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3) Py_RETURN_NONE;
  return guarded([&]() -> PyObject* {
    const at::Tensor* codes = plain(args[0], at::kByte, 2);
    if (!codes || !codes->is_contiguous()) return nullptr;
    const int64_t rows = codes->size(0), k = 2 * codes->size(1);
    if (rows <= 0 || k <= 0 || k % 16 != 0) return nullptr;
    const at::Tensor* scales = matrix(args[1], at::kByte, rows, k / 16);
    float* s32;
    if (!scales || !scale_arg(args[2], &s32)) return nullptr;
    const uint8_t *cp = bytes(*codes), *sp = bytes(*scales);
    const c10::Device dev = codes->device();
    at::Tensor out;
    int st;
    {
      const WithoutGil released;
      out = empty({rows, k}, at::kFloat, dev);
      st = mixfp4_dequantize(cp, sp, s32, rows, k, floats(out), stream_of(dev));
    }
    return st == MIXFP4_OK ? THPVariable_Wrap(out) : nullptr;
  });
}

PyMethodDef kMethods[] = {
    {"quantize", reinterpret_cast<PyCFunction>(quantize), METH_FASTCALL, nullptr},
    {"gemm", reinterpret_cast<PyCFunction>(gemm), METH_FASTCALL, nullptr},
    {"decode_step", reinterpret_cast<PyCFunction>(decode_step), METH_FASTCALL, nullptr},
    {"dequantize", reinterpret_cast<PyCFunction>(dequantize), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_native",
                       "Native call path of the MixFP4 binding.", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&kModule); }
