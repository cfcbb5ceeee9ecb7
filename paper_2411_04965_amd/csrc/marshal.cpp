// Argument marshalling of the linears a serving loop calls most, as a Python module.  The same calls through ctypes cost 2.4 us
// of host time each beside the launches (3.5 us more where workspace and output are allocated), and small layers are bound
// by the host.  Here plain tensors are unpacked directly: 0.7 us, and 1.5 us for both allocations.
//
// A function takes only what it can pass on as it stands -- exact tensors (no subclass, no torch-function mode), contiguous
// input on a GPU, float32 or bfloat16, plain ints and floats -- and returns None for anything else before it has done
// anything: the caller then goes the general way, which also words the errors.  Otherwise it returns the output, or the
// library's status where that is not 0.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/bitlinear.h"

namespace {

// the library's functions, handed over by the binding that loaded it (so two copies of this package in one process keep apart)
struct {
  decltype(&::bitlinear_a4) a4;
  decltype(&::bitlinear_a8_sparse) a8_sparse;
  decltype(&::bitlinear_a4_gate_up) gate_up;
  decltype(&::bitlinear_workspace_bytes) workspace_bytes;
  decltype(&::bitlinear_gate_up_workspace_bytes) gate_up_workspace_bytes;
} lib;

PyObject* get_device = nullptr;    // torch._C._cuda_getDevice
PyObject* get_stream = nullptr;    // torch._C._cuda_getCurrentRawStream
PyObject* str_H = nullptr;

struct NotPlain {};

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw NotPlain();
  return THPVariable_Unpack(o);
}

void* pointer(PyObject* o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }

int dtype_code(at::ScalarType t) {
  if (t == at::kFloat) return BL_F32;
  if (t == at::kBFloat16) return BL_BF16;
  throw NotPlain();
}

int64_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw NotPlain();
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow) throw NotPlain();
  return v;
}

float real(PyObject* o) {
  if (!PyFloat_CheckExact(o)) throw NotPlain();
  return (float)PyFloat_AS_DOUBLE(o);
}

bool truth(PyObject* o) {
  if (!PyBool_Check(o)) throw NotPlain();
  return o == Py_True;
}

// the raw handle of the current stream of the current device
void* stream() {
  PyObject* d = PyObject_CallNoArgs(get_device);
  if (!d) throw std::exception_ptr();
  PyObject* s = PyObject_CallOneArg(get_stream, d);
  Py_DECREF(d);
  if (!s) throw std::exception_ptr();
  void* p = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  if (!p && PyErr_Occurred()) throw std::exception_ptr();
  return p;
}

struct Input {
  const at::Tensor& x;
  int dt;
  int64_t M, K;
  void* p;
  explicit Input(PyObject* o) : x(tensor(o)) {
    if (!x.is_cuda() || x.dim() != 2 || !x.is_contiguous()) throw NotPlain();
    dt = dtype_code(x.scalar_type());
    M = x.size(0);
    K = x.size(1);
    p = x.data_ptr();
  }
};

// a caller's workspace, or one of `bytes` (asked for only then) that lives until this object goes
struct Workspace {
  at::Tensor own;
  void* p = nullptr;
  size_t n = 0;
  template <typename F>
  Workspace(PyObject* o, const Input& in, F bytes) {
    if (o != Py_None) {
      const at::Tensor& t = tensor(o);
      p = t.data_ptr();
      n = (size_t)t.numel();
    } else {
      n = bytes();
      if (n < 16) n = 16;
      own = at::empty({(int64_t)n}, in.x.options().dtype(at::kByte).requires_grad(false));
      p = own.data_ptr();
    }
  }
};

struct Output {
  at::Tensor own;
  PyObject* given = nullptr;
  void* p = nullptr;
  int dt = 0;
  Output(PyObject* out, const Input& in, int64_t N, at::ScalarType type) {
    if (out != Py_None) {
      const at::Tensor& t = tensor(out);
      given = out;
      dt = dtype_code(t.scalar_type());
      p = t.data_ptr();
    } else {
      dt = dtype_code(type);
      own = at::empty({in.M, N}, in.x.options().dtype(type).requires_grad(false));
      p = own.data_ptr();
    }
  }
  PyObject* result() noexcept {
    if (!given) return THPVariable_Wrap(std::move(own));
    Py_INCREF(given);
    return given;
  }
};

at::ScalarType scalar_type(PyObject* o) {
  if (!THPDtype_Check(o)) throw NotPlain();
  return reinterpret_cast<THPDtype*>(o)->scalar_type;
}

bool mx(int64_t layout) { return layout == BL_W_MX4 || layout == BL_W_MX2; }

template <typename F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F body) {
  try {
    if (n != want || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    return body();
  } catch (const NotPlain&) {
    Py_RETURN_NONE;
  } catch (const std::exception_ptr&) {
    return nullptr;                                        // (a Python error is set)
  } catch (python_error& e) {                              // (Python code that torch called, a dispatch mode for instance: its own error)
    e.restore();
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
  } catch (const std::exception&) {                        // (allocation, a tensor without storage: nothing is enqueued yet,
    if (PyErr_Occurred()) return nullptr;                  //  and the general way meets the same and words it)
    Py_RETURN_NONE;
  }
}

// (X, W_packed, alpha, N, eps, act_fp4, y_dtype, ws, out, layout)
PyObject* a4(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&]() -> PyObject* {
    const Input in(a[0]);
    void* const w = pointer(a[1]);
    const float* const alpha = (const float*)pointer(a[2]);
    const int64_t N = integer(a[3]), layout = integer(a[9]);
    const float eps = real(a[4]);
    const bool fp4 = truth(a[5]);
    if (in.M < 1 || N < 1 || N > ((int64_t)1 << 31) || layout < 0 || layout > 4) throw NotPlain();
    const int mode = fp4 ? (mx(layout) ? BL_ACT_FP4_E2M1_B32_MX : BL_ACT_FP4_E2M1_B32)
                         : (mx(layout) ? BL_ACT_INT4_ABSMEAN_MX6 : BL_ACT_INT4_ABSMEAN);
    Workspace ws(a[7], in, [&] { return lib.workspace_bytes((bl_act_mode)mode, in.M, N, in.K); });
    Output y(a[8], in, N, scalar_type(a[6]));
    void* const s = stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = lib.a4(in.p, (bl_dtype)in.dt, in.M, in.K, w, (bl_w_layout)layout, alpha, N, eps, fp4 ? 1 : 0, y.p,
                      (bl_dtype)y.dt, nullptr, ws.p, ws.n, s);
    Py_END_ALLOW_THREADS
    return rc ? PyLong_FromLong(rc) : y.result();
  });
}

// (X, topk, W_packed, alpha, N, eps, layout, y_dtype, ws, out)
PyObject* a8_sparse(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&]() -> PyObject* {
    const Input in(a[0]);
    const int64_t topk = integer(a[1]), N = integer(a[4]), layout = integer(a[6]);
    void* const w = pointer(a[2]);
    const float* const alpha = (const float*)pointer(a[3]);
    const float eps = real(a[5]);
    if (in.M < 1 || N < 1 || N > ((int64_t)1 << 31) || layout < 0 || layout > 4) throw NotPlain();
    Workspace ws(a[8], in, [&] { return lib.workspace_bytes(BL_ACT_TOPK_INT8_ABSMAX, in.M, N, in.K); });
    Output y(a[9], in, N, scalar_type(a[7]));
    void* const s = stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = lib.a8_sparse(in.p, (bl_dtype)in.dt, in.M, in.K, topk, w, (bl_w_layout)layout, alpha, N, eps, y.p,
                             (bl_dtype)y.dt, nullptr, ws.p, ws.n, s);
    Py_END_ALLOW_THREADS
    return rc ? PyLong_FromLong(rc) : y.result();
  });
}

// (X, W_gate, alpha_gate, W_up, alpha_up, N, eps, layout, want, ws, out): want == ("H",), out None or {"H": tensor}
PyObject* gate_up(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    PyObject* const want = a[8];
    if (!PyTuple_CheckExact(want) || PyTuple_GET_SIZE(want) != 1 || !PyUnicode_CheckExact(PyTuple_GET_ITEM(want, 0)) ||
        PyUnicode_Compare(PyTuple_GET_ITEM(want, 0), str_H) != 0)
      throw NotPlain();
    PyObject* h = Py_None;
    if (a[10] != Py_None) {
      if (!PyDict_CheckExact(a[10]) || PyDict_GET_SIZE(a[10]) > 1) throw NotPlain();
      h = PyDict_GetItemWithError(a[10], str_H);           // (borrowed)
      if (!h || h == Py_None) { PyErr_Clear(); throw NotPlain(); }
    }
    const Input in(a[0]);
    void* const wg = pointer(a[1]);
    const float* const ag = (const float*)pointer(a[2]);
    void* const wu = pointer(a[3]);
    const float* const au = (const float*)pointer(a[4]);
    const int64_t N = integer(a[5]), layout = integer(a[7]);
    const float eps = real(a[6]);
    if (in.M < 1 || N < 1 || N > ((int64_t)1 << 31) || layout < 0 || layout > 4) throw NotPlain();
    Workspace ws(a[9], in, [&] { return lib.gate_up_workspace_bytes(in.M, N, in.K, (bl_w_layout)layout); });
    void* hp;
    at::Tensor own;
    if (h != Py_None) {
      hp = tensor(h).data_ptr();
    } else {
      own = at::empty({in.M, N}, in.x.options().dtype(at::kBFloat16).requires_grad(false));
      hp = own.data_ptr();
    }
    void* const s = stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = lib.gate_up(in.p, (bl_dtype)in.dt, in.M, in.K, wg, ag, wu, au, (bl_w_layout)layout, N, eps, nullptr, nullptr,
                              BL_F32, hp, ws.p, ws.n, s);
    Py_END_ALLOW_THREADS
    if (rc) return PyLong_FromLong(rc);
    PyObject* const r = PyDict_New();
    if (!r) return nullptr;
    PyObject* const v = h != Py_None ? (Py_INCREF(h), h) : THPVariable_Wrap(std::move(own));
    const int bad = v ? PyDict_SetItem(r, str_H, v) : -1;
    Py_XDECREF(v);
    if (bad) { Py_DECREF(r); return nullptr; }
    return r;
  });
}

// (addresses of bitlinear_a4, bitlinear_a8_sparse, bitlinear_a4_gate_up, bitlinear_workspace_bytes, bitlinear_gate_up_workspace_bytes)
PyObject* use(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* p[5];
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "five addresses expected");
    return nullptr;
  }
  for (int i = 0; i < 5; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  lib = {(decltype(lib.a4))p[0], (decltype(lib.a8_sparse))p[1], (decltype(lib.gate_up))p[2], (decltype(lib.workspace_bytes))p[3],
         (decltype(lib.gate_up_workspace_bytes))p[4]};
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"use", (PyCFunction)(void (*)(void))use, METH_FASTCALL, "the library's functions, by address; before any other call"},
    {"a4", (PyCFunction)(void (*)(void))a4, METH_FASTCALL, "bitlinear_a4"},
    {"a8_sparse", (PyCFunction)(void (*)(void))a8_sparse, METH_FASTCALL, "bitlinear_a8_sparse"},
    {"gate_up", (PyCFunction)(void (*)(void))gate_up, METH_FASTCALL, "bitlinear_a4_gate_up, H only"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "bitlinear_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_bitlinear_marshal() {
  PyObject* const c = PyImport_ImportModule("torch._C");
  if (!c) return nullptr;
  get_device = PyObject_GetAttrString(c, "_cuda_getDevice");
  get_stream = get_device ? PyObject_GetAttrString(c, "_cuda_getCurrentRawStream") : nullptr;
  Py_DECREF(c);
  if (!get_stream) {
    if (PyErr_Occurred()) PyErr_Clear();
    PyErr_SetString(PyExc_ImportError, "torch without GPU support");
    return nullptr;
  }
  str_H = PyUnicode_InternFromString("H");
  return str_H ? PyModule_Create(&module) : nullptr;
}
