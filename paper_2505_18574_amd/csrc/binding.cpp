// Native side of ops.py: reads the tensors and calls the C ABI (include/ac.h) in one step.
//
// On this path a launch takes the GPU no longer than argument checks in Python take the host: of the 6.6 us that a call
// of a few-microsecond kernel cost there, 2.6 are the runtime's launch; through these functions a call is 3.4 us.
//
// Every function takes the arguments of its namesake in ops.py, all of them, in order, and returns the ac_status of the
// call, or PYTHON where an argument is not of the plain kind that is read here (an exact torch.Tensor of the right type,
// shape and device, an int of 32 bits, a bool, ...): ops.py then does the call with its own checks, which accept what is
// unusual and raise what is wrong.  Nothing is kept from one call to the next.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

#include "../../include/ac.h"

namespace {

constexpr long PYTHON = 1;  // no ac_status: those are zero or negative

// Thrown by the readers below and caught in call(): the argument is not plain.
struct NotPlain {};
void require(bool ok) {
  if (!ok) throw NotPlain{};
}

const at::Tensor& tensor(PyObject* o, at::ScalarType type, int64_t dims) {
  require(THPVariable_CheckExact(o));
  const at::Tensor& t = THPVariable_Unpack(o);
  require(t.defined() && t.scalar_type() == type && t.dim() == dims && t.is_cuda() && t.layout() == at::kStrided);
  return t;
}
const at::Tensor& dense(PyObject* o, at::ScalarType type, int64_t dims) {
  const at::Tensor& t = tensor(o, type, dims);
  require(t.is_contiguous());
  return t;
}
int32_t narrow(int64_t v) {
  require(v >= INT32_MIN && v <= INT32_MAX);
  return (int32_t)v;
}
int32_t integer(PyObject* o) {
  require(PyLong_Check(o));
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  require(overflow == 0);
  return narrow(v);
}
bool boolean(PyObject* o) {
  require(o == Py_True || o == Py_False);
  return o == Py_True;
}
float real(PyObject* o) {
  require(PyFloat_Check(o));
  return (float)PyFloat_AS_DOUBLE(o);
}
void* stream_of(PyObject* o) {
  if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream().stream();
  PyObject* handle = PyObject_GetAttrString(o, "cuda_stream");
  void* s = handle != nullptr && PyLong_Check(handle) ? PyLong_AsVoidPtr(handle) : nullptr;
  const bool ok = handle != nullptr && PyLong_Check(handle) && !PyErr_Occurred();
  Py_XDECREF(handle);
  PyErr_Clear();
  require(ok);
  return s;
}

struct Matrix {  // 2-D, row-major
  void* data;
  int64_t rows, cols, pitch;
};
Matrix matrix(PyObject* o, at::ScalarType type) {
  const at::Tensor& t = tensor(o, type, 2);
  const Matrix m = {t.data_ptr(), t.size(0), t.size(1), t.stride(0)};
  require(m.cols <= 1 || t.stride(1) == 1);
  return m;
}
struct Workspace {
  void* data = nullptr;
  size_t bytes = 0;
};
Workspace workspace_of(PyObject* o) {
  Workspace w;
  if (o != Py_None) {
    require(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    require(t.defined() && t.layout() == at::kStrided);
    w.data = t.data_ptr(), w.bytes = t.nbytes();
  }
  return w;
}
struct Bias {
  const int32_t* data = nullptr;
  int64_t pitch = 0;
};
// None, a row of N values or an M x N matrix
Bias bias_of(PyObject* o, int64_t M, int64_t N) {
  Bias b;
  if (o != Py_None) {
    require(THPVariable_CheckExact(o));
    const int64_t dims = THPVariable_Unpack(o).dim();
    const at::Tensor& t = tensor(o, at::kInt, dims);
    if (dims == 2) {
      require(t.size(0) == M && t.size(1) == N && t.stride(1) == 1);
      b.pitch = t.stride(0);
    } else {
      require(dims == 1 && t.size(0) == N && (N <= 1 || t.stride(0) == 1));
    }
    b.data = (const int32_t*)t.data_ptr();
  }
  return b;
}
float* optional(PyObject* o, int64_t dims, int64_t a, int64_t b, int64_t c = 0) {  // None or dense fp32 [a][b] or [a][b][c]
  if (o == Py_None) return nullptr;
  const at::Tensor& t = dense(o, at::kFloat, dims);
  require(t.size(0) == a && t.size(1) == b && (dims < 3 || t.size(2) == c));
  return (float*)t.data_ptr();
}

// Runs f(args), which reads the arguments and returns a callable that makes the C call; that one runs without the GIL.
template <int NARGS, class F>
PyObject* call(PyObject* const* args, Py_ssize_t nargs, F f) {
  long status = PYTHON;
  try {
    if (nargs == NARGS && !at::impl::torch_function_mode_enabled()) {
      const auto launch = f(args);
      Py_BEGIN_ALLOW_THREADS
      status = (long)launch();
      Py_END_ALLOW_THREADS
    }
  } catch (...) {  // not plain, or a tensor without memory: Python says what is wrong
    PyErr_Clear();
    status = PYTHON;
  }
  return PyLong_FromLong(status);
}

struct GemmI8 {
  Matrix A, B, C;
  Bias bias;
  int32_t M, N, K;
};
GemmI8 gemm_i8_operands(PyObject* const* a, bool ta, bool tb, at::ScalarType out) {
  GemmI8 g;
  g.A = matrix(a[0], at::kChar), g.B = matrix(a[1], at::kChar), g.C = matrix(a[3], out);
  const int64_t M = ta ? g.A.cols : g.A.rows, K = ta ? g.A.rows : g.A.cols, N = tb ? g.B.rows : g.B.cols;
  require((tb ? g.B.cols : g.B.rows) == K && g.C.rows == M && g.C.cols == N);
  g.M = narrow(M), g.N = narrow(N), g.K = narrow(K);
  return g;
}

PyObject* gemm_i8(PyObject*, PyObject* const* args, Py_ssize_t nargs) {  // A, B, bias, C, shift, act, workspace, stream
  return call<8>(args, nargs, [](PyObject* const* a) {
    GemmI8 g = gemm_i8_operands(a, false, false, at::kChar);
    g.bias = bias_of(a[2], g.M, g.N);
    const int32_t shift = integer(a[4]), act = integer(a[5]);
    const Workspace w = workspace_of(a[6]);
    void* s = stream_of(a[7]);
    return [=] {
      return ac_gemm_i8((const int8_t*)g.A.data, g.A.pitch, (const int8_t*)g.B.data, g.B.pitch, g.bias.data, g.bias.pitch,
                        (int8_t*)g.C.data, g.C.pitch, g.M, g.N, g.K, shift, act, w.data, w.bytes, s);
    };
  });
}

PyObject* gemm_i8_t(PyObject*, PyObject* const* args, Py_ssize_t nargs) {  // A, B, bias, C, shift, act, trans_a, trans_b, stream
  return call<9>(args, nargs, [](PyObject* const* a) {
    const bool ta = boolean(a[6]), tb = boolean(a[7]);
    GemmI8 g = gemm_i8_operands(a, ta, tb, at::kChar);
    g.bias = bias_of(a[2], g.M, g.N);
    const int32_t shift = integer(a[4]), act = integer(a[5]);
    void* s = stream_of(a[8]);
    return [=] {
      return ac_gemm_i8_t((const int8_t*)g.A.data, g.A.pitch, (const int8_t*)g.B.data, g.B.pitch, g.bias.data, g.bias.pitch,
                          (int8_t*)g.C.data, g.C.pitch, g.M, g.N, g.K, shift, act, ta, tb, s);
    };
  });
}

PyObject* gemm_i8_acc32(PyObject*, PyObject* const* args, Py_ssize_t nargs) {  // A, B, bias, C, stream
  return call<5>(args, nargs, [](PyObject* const* a) {
    GemmI8 g = gemm_i8_operands(a, false, false, at::kInt);
    g.bias = bias_of(a[2], g.M, g.N);
    void* s = stream_of(a[4]);
    return [=] {
      return ac_gemm_i8_acc32((const int8_t*)g.A.data, g.A.pitch, (const int8_t*)g.B.data, g.B.pitch, g.bias.data, g.bias.pitch,
                              (int32_t*)g.C.data, g.C.pitch, g.M, g.N, g.K, s);
    };
  });
}

PyObject* conv2d_i8(PyObject*, PyObject* const* args, Py_ssize_t nargs) {  // x, w, bias, out, stride, pad, shift, act, workspace, stream
  return call<10>(args, nargs, [](PyObject* const* a) {
    const at::Tensor &x = dense(a[0], at::kChar, 4), &w = dense(a[1], at::kChar, 4), &out = dense(a[3], at::kChar, 4);
    const int32_t Nb = narrow(x.size(0)), H = narrow(x.size(1)), W = narrow(x.size(2)), Cin = narrow(x.size(3));
    const int32_t KH = narrow(w.size(0)), KW = narrow(w.size(1)), Cout = narrow(w.size(3));
    const int32_t stride = integer(a[4]), pad = integer(a[5]), shift = integer(a[6]), act = integer(a[7]);
    const int64_t oh = (int64_t)H + 2 * (int64_t)pad - KH, ow = (int64_t)W + 2 * (int64_t)pad - KW;
    require(w.size(2) == Cin && stride >= 1 && oh >= 0 && ow >= 0);
    require(out.size(0) == Nb && out.size(1) == oh / stride + 1 && out.size(2) == ow / stride + 1 && out.size(3) == Cout);
    const int32_t* bias = nullptr;
    if (a[2] != Py_None) {
      const at::Tensor& b = dense(a[2], at::kInt, 1);
      require(b.size(0) == Cout);
      bias = (const int32_t*)b.data_ptr();
    }
    const Workspace ws = workspace_of(a[8]);
    void* s = stream_of(a[9]);
    const int8_t *xp = (const int8_t*)x.data_ptr(), *wp = (const int8_t*)w.data_ptr();
    int8_t* op = (int8_t*)out.data_ptr();
    return [=] { return ac_conv2d_i8(xp, wp, bias, op, Nb, H, W, Cin, Cout, KH, KW, stride, pad, shift, act, ws.data, ws.bytes, s); };
  });
}

PyObject* gemm_bf16_ws(PyObject*, PyObject* const* args, Py_ssize_t nargs) {  // A, B, C, alpha, beta, workspace, stream
  return call<7>(args, nargs, [](PyObject* const* a) {
    const Matrix A = matrix(a[0], at::kBFloat16), B = matrix(a[1], at::kBFloat16), C = matrix(a[2], at::kFloat);
    require(B.rows == A.cols && C.rows == A.rows && C.cols == B.cols);
    const int32_t M = narrow(A.rows), N = narrow(B.cols), K = narrow(A.cols);
    const float alpha = real(a[3]), beta = real(a[4]);
    const Workspace w = workspace_of(a[5]);
    void* s = stream_of(a[6]);
    return [=] {
      return ac_gemm_bf16_ws((const uint16_t*)A.data, A.pitch, (const uint16_t*)B.data, B.pitch, (float*)C.data, C.pitch, M, N, K, alpha, beta, w.data, w.bytes, s);
    };
  });
}

PyObject* batched_gemm_f32(PyObject*, PyObject* const* args, Py_ssize_t nargs) {  // A, B, C, x, d, y, stream
  return call<7>(args, nargs, [](PyObject* const* a) {
    const at::Tensor& A = dense(a[0], at::kFloat, 3);
    const int64_t batch = A.size(0), n = A.size(1);
    require(A.size(2) == n && a[1] != Py_None);
    const float *Ap = (const float*)A.data_ptr(), *Bp = optional(a[1], 3, batch, n, n);
    float *C = optional(a[2], 3, batch, n, n), *y = optional(a[5], 2, batch, n);
    const float *x = optional(a[3], 2, batch, n), *d = optional(a[4], 2, batch, n);
    const int32_t n32 = narrow(n);
    void* s = stream_of(a[6]);
    return [=] { return ac_batched_gemm_f32(Ap, Bp, C, x, d, y, n32, batch, s); };
  });
}

PyObject* tinympc_forward_f32(PyObject*, PyObject* const* args, Py_ssize_t nargs) {  // Adyn, Bdyn, Kinf, x0, d, u, x_out, stream
  return call<8>(args, nargs, [](PyObject* const* a) {
    for (int i = 0; i < 6; i++) require(a[i] != Py_None);
    const at::Tensor &B = dense(a[1], at::kFloat, 2), &d = dense(a[4], at::kFloat, 3);
    const int64_t nx = B.size(0), nu = B.size(1), batch = d.size(0), horizon = d.size(1);
    const float *Ap = optional(a[0], 2, nx, nx), *Bp = (const float*)B.data_ptr(), *Kp = optional(a[2], 2, nu, nx), *x0 = optional(a[3], 2, batch, nx);
    const float* dp = optional(a[4], 3, batch, horizon, nu);
    float *u = optional(a[5], 3, batch, horizon, nu), *x = optional(a[6], 3, batch, horizon + 1, nx);
    const int32_t nx32 = narrow(nx), nu32 = narrow(nu), h32 = narrow(horizon);
    void* s = stream_of(a[7]);
    return [=] { return ac_tinympc_forward_f32(Ap, Bp, Kp, x0, dp, u, x, nx32, nu32, h32, batch, s); };
  });
}

#define AC_METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {AC_METHOD(gemm_i8), AC_METHOD(gemm_i8_t), AC_METHOD(gemm_i8_acc32), AC_METHOD(conv2d_i8), AC_METHOD(gemm_bf16_ws),
                         AC_METHOD(batched_gemm_f32), AC_METHOD(tinympc_forward_f32), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
