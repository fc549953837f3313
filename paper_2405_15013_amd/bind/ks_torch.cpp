// Native form of the binding's matmul() and chain() (the module _ks_torch).
//
// Both functions take the arguments of their Python namesakes, check them, and
// call libks.so on plain tensors.  Whatever is not plain -- a wrong size, type
// or device, a tensor subclass, an active dispatch mode, transform or trace, a
// status other than KS_OK -- returns None with nothing enqueued, and the Python
// code runs the call from the start (and reports the error, if it is one).
//
// A call of matmul() spent 9.3 us on the host, of which the launch 2.4:
// 2.6 in torch.cuda.current_stream(), 1.4 in torch.empty(), the rest in attribute
// lookups and ctypes; this way it takes 4.6 (3.6 with `out`), and chain() of ten
// factors 11 instead of 26.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <string>

#include "../../include/ks.h"

namespace {

decltype(&ks_matmul) p_matmul = nullptr;
decltype(&ks_matmul_bias_act) p_matmul_bias_act = nullptr;
decltype(&ks_chain) p_chain = nullptr;
decltype(&ks_chain_workspace_bytes) p_chain_workspace_bytes = nullptr;
PyObject* f_device = nullptr;  // torch._C._cuda_getDevice
PyObject* f_stream = nullptr;  // torch._C._cuda_getCurrentRawStream

// No mode, transform or trace that a torch call would have to go through.
bool plain_state() {
  return !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled() &&
         !torch::jit::tracer::isTracing() &&
         !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) &&
         !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::Functionalize) &&
         !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::PythonDispatcher);
}

// A dense contiguous device tensor with memory of its own, of no subclass.
const at::Tensor* plain_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  static const c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot,
                                            c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                            c10::DispatchKey::Batched, c10::DispatchKey::Functionalize,
                                            c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                            c10::DispatchKey::ZeroTensor});
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.is_quantized() || !t.has_storage() ||
      t.key_set().has_any(wrapped) || !t.is_contiguous())
    return nullptr;
  return &t;
}

int dtype_code(at::ScalarType t) {
  switch (t) {
    case at::kFloat: return KS_F32;
    case at::kBFloat16: return KS_BF16;
    case at::kHalf: return KS_F16;
    case at::kFloat8_e4m3fn: return KS_FP8_E4M3;
    default: return -1;
  }
}

int layout_code(PyObject* o) {
  if (!PyUnicode_CheckExact(o)) return -1;
  if (PyUnicode_CompareWithASCIIString(o, "bsl") == 0) return KS_LAYOUT_BSL;
  if (PyUnicode_CompareWithASCIIString(o, "bsf") == 0) return KS_LAYOUT_BSF;
  return -1;
}

// Four positive sizes whose products stay far from overflow.
bool pattern_of(PyObject* o, int64_t (&p)[4]) {
  if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 4) return false;
  for (int q = 0; q < 4; ++q) {
    PyObject* v = PyTuple_GET_ITEM(o, q);
    if (!PyLong_CheckExact(v)) return false;
    int overflow = 0;
    p[q] = PyLong_AsLongLongAndOverflow(v, &overflow);
    if (overflow || p[q] < 1 || p[q] > 1 << 15) return false;
  }
  return true;
}

// The current stream of the current device (as the Python code takes it).
bool current_stream(void** s) {
  PyObject* dev = PyObject_CallNoArgs(f_device);
  PyObject* st = dev ? PyObject_CallOneArg(f_stream, dev) : nullptr;
  Py_XDECREF(dev);
  if (st) *s = PyLong_AsVoidPtr(st);
  const bool ok = st && !PyErr_Occurred();
  Py_XDECREF(st);
  if (!ok) PyErr_Clear();
  return ok;
}

// Batch of X for width N (0 and less: not a shape the call takes).
int64_t batch_of(const at::Tensor& x, int64_t N, int layout) {
  const int64_t n = x.numel();
  if (n % N) return -1;
  const int64_t batch = n / N;
  if (x.dim() == 1) return batch;
  if (x.dim() != 2) return -1;
  return x.size(layout == KS_LAYOUT_BSF ? 0 : 1) == batch && x.size(layout == KS_LAYOUT_BSF ? 1 : 0) == N ? batch : -1;
}

// The interpreter lock, let go for as long as this lives (an allocation may wait
// for another thread that needs it).
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// `given` if it is a fitting output, a new tensor if it is None, else nothing.
at::Tensor output(PyObject* given, int64_t r, int64_t c, at::ScalarType dtype, const at::Tensor& x) {
  if (given == Py_None) {
    Unlocked u;
    return at::empty({r, c}, at::TensorOptions().dtype(dtype).device(x.device()));
  }
  const at::Tensor* o = plain_tensor(given);
  if (!o || o->scalar_type() != dtype || o->device() != x.device() || o->numel() != r * c ||
      (o->dim() == 2 && (o->size(0) != r || o->size(1) != c)))
    return at::Tensor();
  return *o;
}

PyObject* result(PyObject* given, const at::Tensor& y) {
  if (given == Py_None) return THPVariable_Wrap(y);
  Py_INCREF(given);
  return given;
}

// matmul(X, K_values, pattern, layout, out, bias, act)
PyObject* fast_matmul(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 7 || !p_matmul || !plain_state()) Py_RETURN_NONE;
  try {
    int64_t p[4];
    const at::Tensor *x = plain_tensor(a[0]), *k = plain_tensor(a[1]), *bias = nullptr;
    const int layout = layout_code(a[3]);
    if (!x || !k || layout < 0 || !pattern_of(a[2], p)) Py_RETURN_NONE;
    const int dtype = dtype_code(x->scalar_type());
    const int64_t N = p[0] * p[2] * p[3], M = p[0] * p[1] * p[3];
    if (dtype < 0 || k->scalar_type() != x->scalar_type() || k->device() != x->device() || k->numel() != M * p[2])
      Py_RETURN_NONE;
    const int64_t batch = batch_of(*x, N, layout);
    if (batch < 0) Py_RETURN_NONE;
    const at::ScalarType ydtype = dtype == KS_FP8_E4M3 ? at::kBFloat16 : x->scalar_type();
    int act = KS_ACT_NONE;
    if (a[6] != Py_None) {
      if (!PyUnicode_CheckExact(a[6]) || PyUnicode_CompareWithASCIIString(a[6], "gelu") != 0) Py_RETURN_NONE;
      act = KS_ACT_GELU;
    }
    if (a[5] != Py_None) {
      bias = plain_tensor(a[5]);
      if (!bias || bias->scalar_type() != ydtype || bias->device() != x->device() || bias->numel() != M) Py_RETURN_NONE;
    }
    void* stream = nullptr;
    if (!current_stream(&stream)) Py_RETURN_NONE;
    const bool bsf = layout == KS_LAYOUT_BSF;
    const at::Tensor y = output(a[4], bsf ? batch : M, bsf ? M : batch, ydtype, *x);
    if (!y.defined()) Py_RETURN_NONE;
    const void *kp = k->const_data_ptr(), *xp = x->const_data_ptr(), *bp = bias ? bias->const_data_ptr() : nullptr;
    void* yp = y.data_ptr();
    ks_status_t st;
    {
      Unlocked u;
      st = bias || act != KS_ACT_NONE
               ? p_matmul_bias_act(p[0], p[1], p[2], p[3], kp, bp, act, xp, yp, batch, layout, dtype, stream)
               : p_matmul(p[0], p[1], p[2], p[3], kp, xp, yp, batch, layout, dtype, stream);
    }
    if (st != KS_OK) Py_RETURN_NONE;
    return result(a[4], y);
  } catch (const std::exception&) {
    Py_RETURN_NONE;  // (an allocation that failed, say: the Python code meets it again)
  }
}

// chain(X, factors, layout, out, workspace)
PyObject* fast_chain(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 5 || !p_chain || !plain_state()) Py_RETURN_NONE;
  try {
    constexpr Py_ssize_t kMax = 32;
    const at::Tensor *x = plain_tensor(a[0]), *given_ws = nullptr;
    const int layout = layout_code(a[2]);
    const bool list = PyList_CheckExact(a[1]);
    if (!x || layout < 0 || (!list && !PyTuple_CheckExact(a[1]))) Py_RETURN_NONE;
    const Py_ssize_t nf = list ? PyList_GET_SIZE(a[1]) : PyTuple_GET_SIZE(a[1]);
    if (nf < 1 || nf > kMax) Py_RETURN_NONE;
    const int dtype = dtype_code(x->scalar_type());
    if (dtype < 0) Py_RETURN_NONE;
    ks_factor_t f[kMax];
    for (Py_ssize_t q = 0; q < nf; ++q) {
      PyObject* pair = list ? PyList_GET_ITEM(a[1], q) : PyTuple_GET_ITEM(a[1], q);
      int64_t p[4];
      if (!PyTuple_CheckExact(pair) || PyTuple_GET_SIZE(pair) != 2 || !pattern_of(PyTuple_GET_ITEM(pair, 0), p))
        Py_RETURN_NONE;
      const at::Tensor* k = plain_tensor(PyTuple_GET_ITEM(pair, 1));
      if (!k || k->scalar_type() != x->scalar_type() || k->device() != x->device() ||
          k->numel() != p[0] * p[1] * p[2] * p[3])
        Py_RETURN_NONE;
      if (q > 0 && f[q - 1].a * f[q - 1].c * f[q - 1].d != p[0] * p[1] * p[3]) Py_RETURN_NONE;
      f[q] = ks_factor_t{p[0], p[1], p[2], p[3], k->const_data_ptr()};
    }
    const int64_t N = f[nf - 1].a * f[nf - 1].c * f[nf - 1].d, M = f[0].a * f[0].b * f[0].d;
    const int64_t batch = batch_of(*x, N, layout);
    if (batch < 0) Py_RETURN_NONE;
    const size_t need = p_chain_workspace_bytes(f, (int)nf, batch, dtype);
    at::Tensor ws;
    size_t have = 0;
    if (a[4] != Py_None) {
      given_ws = plain_tensor(a[4]);
      if (!given_ws || given_ws->device() != x->device()) Py_RETURN_NONE;
      ws = *given_ws;
      have = (size_t)ws.numel() * ws.element_size();
    } else if (need > 0) {
      Unlocked u;
      ws = at::empty({(int64_t)need}, at::TensorOptions().dtype(at::kByte).device(x->device()));
      have = need;
    }
    void* stream = nullptr;
    if (!current_stream(&stream)) Py_RETURN_NONE;
    const bool bsf = layout == KS_LAYOUT_BSF;
    const at::Tensor y = output(a[3], bsf ? batch : M, bsf ? M : batch, x->scalar_type(), *x);
    if (!y.defined()) Py_RETURN_NONE;
    const void* xp = x->const_data_ptr();
    void *yp = y.data_ptr(), *wp = ws.defined() ? ws.data_ptr() : nullptr;
    ks_status_t st;
    {
      Unlocked u;
      st = p_chain(f, (int)nf, xp, yp, batch, layout, dtype, wp, have, stream);
    }
    if (st != KS_OK) Py_RETURN_NONE;
    return result(a[3], y);
  } catch (const std::exception&) {
    Py_RETURN_NONE;
  }
}

// The PyTorch whose class layouts are compiled in.
const char built_for[] = "built for PyTorch " KS_TORCH_VERSION ";";

// init({name: address of the libks.so function}, _cuda_getDevice, _cuda_getCurrentRawStream,
// torch.__version__)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 4 || !PyDict_Check(a[0]) || !PyUnicode_Check(a[3])) {
    PyErr_SetString(PyExc_TypeError, "init(addresses, device, stream, version)");
    return nullptr;
  }
  const char* version = PyUnicode_AsUTF8(a[3]);
  if (!version) return nullptr;
  if ("built for PyTorch " + std::string(version) + ";" != built_for) {
    PyErr_Format(PyExc_ImportError, "_ks_torch was %s this is %U", built_for, a[3]);
    return nullptr;
  }
  auto address = [&](const char* name) -> void* {
    PyObject* v = PyDict_GetItemString(a[0], name);
    return v ? PyLong_AsVoidPtr(v) : nullptr;
  };
  p_matmul = reinterpret_cast<decltype(p_matmul)>(address("ks_matmul"));
  p_matmul_bias_act = reinterpret_cast<decltype(p_matmul_bias_act)>(address("ks_matmul_bias_act"));
  p_chain = reinterpret_cast<decltype(p_chain)>(address("ks_chain"));
  p_chain_workspace_bytes = reinterpret_cast<decltype(p_chain_workspace_bytes)>(address("ks_chain_workspace_bytes"));
  if (PyErr_Occurred()) return nullptr;
  if (!p_matmul || !p_matmul_bias_act || !p_chain || !p_chain_workspace_bytes) {
    PyErr_SetString(PyExc_ValueError, "init: a function's address is missing");
    return nullptr;
  }
  Py_INCREF(a[1]);
  Py_INCREF(a[2]);
  Py_XSETREF(f_device, a[1]);
  Py_XSETREF(f_stream, a[2]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"matmul", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fast_matmul)), METH_FASTCALL, nullptr},
    {"chain", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fast_chain)), METH_FASTCALL, nullptr},
    {"init", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(init)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ks_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__ks_torch() { return PyModule_Create(&module); }
