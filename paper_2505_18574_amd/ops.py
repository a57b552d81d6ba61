"""Thin binding over the C ABI of ``libac_mi355x.so`` (see ``include/ac.h``).

Argument marshalling only: every function takes device tensors (PyTorch-ROCm is
used for device memory and streams, nothing else), passes their addresses,
leading dimensions and sizes to the entry point of the same name, and raises
``AcError`` on a non-zero status.  There is no CPU fallback: if the HIP library
has not been built, loading fails with an ImportError.
"""
from __future__ import annotations

import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libac_mi355x.so")

AC_OK = 0
AC_ERR_NULL, AC_ERR_SHAPE, AC_ERR_STRIDE, AC_ERR_SHIFT = -1, -2, -3, -4
AC_ERR_ACT, AC_ERR_ALIAS, AC_ERR_WORKSPACE, AC_ERR_LAUNCH = -5, -6, -7, -8
AC_ERR_PLAN = -9
AC_ACT_NONE, AC_ACT_RELU = 0, 1

# every symbol include/ac.h declares
EXPORTS = ("ac_gemm_i8", "ac_gemm_i8_workspace_bytes", "ac_conv2d_i8", "ac_gemm_bf16", "ac_batched_gemm_f32",
           "ac_tinympc_forward_f32", "ac_gemm_i8_acc32", "ac_gemm_i8_static",
           "ac_gemm_i8_t", "ac_gemm_i8_planned", "ac_conv2d_i8_planned", "ac_gemm_i8_planned_workspace_bytes", "ac_gemm_bf16_planned",
           "ac_gemm_bf16_planned_workspace_bytes", "ac_gemm_bf16_ws", "ac_gemm_bf16_workspace_bytes",
           "ac_gemm_i8_auto_plan", "ac_gemm_bf16_auto_plan",
           "ac_status_string", "ac_version")

_lib = None
_native = None


class AcError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: status {status} ({status_string(status)})")


def lib() -> ctypes.CDLL:
    """The loaded C-ABI library, with argument types declared."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(
                f"{LIB_PATH} is missing: build it with `python -m paper_2505_18574_amd.build` "
                "(or __graft_entry__.build()); there is no fallback path")
        L = ctypes.CDLL(LIB_PATH)
        vp, i64, i32, sz, f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_size_t, ctypes.c_float
        L.ac_gemm_i8.restype = i32
        L.ac_gemm_i8.argtypes = [vp, i64, vp, i64, vp, i64, vp, i64, i32, i32, i32, i32, i32, vp, sz, vp]
        L.ac_gemm_i8_static.restype = i32
        L.ac_gemm_i8_static.argtypes = L.ac_gemm_i8.argtypes[:-3] + [vp]
        L.ac_gemm_i8_workspace_bytes.restype = sz
        L.ac_gemm_i8_workspace_bytes.argtypes = [i32, i32, i32]
        L.ac_conv2d_i8.restype = i32
        L.ac_conv2d_i8.argtypes = [vp, vp, vp, vp, i32, i32, i32, i32, i32, i32, i32, i32, i32, i32, i32, vp, sz, vp]
        L.ac_conv2d_i8_planned.restype = i32
        L.ac_conv2d_i8_planned.argtypes = [vp, vp, vp, vp, i32, i32, i32, i32, i32, i32, i32, i32, i32, i32, i32, vp, sz, i32, i32, vp]
        L.ac_gemm_bf16.restype = i32
        L.ac_gemm_bf16.argtypes = [vp, i64, vp, i64, vp, i64, i32, i32, i32, f32, f32, vp]
        L.ac_batched_gemm_f32.restype = i32
        L.ac_batched_gemm_f32.argtypes = [vp, vp, vp, vp, vp, vp, i32, i64, vp]
        L.ac_gemm_i8_acc32.restype = i32
        L.ac_gemm_i8_acc32.argtypes = [vp, i64, vp, i64, vp, i64, vp, i64, i32, i32, i32, vp]
        L.ac_tinympc_forward_f32.restype = i32
        L.ac_tinympc_forward_f32.argtypes = [vp, vp, vp, vp, vp, vp, vp, i32, i32, i32, i64, vp]
        L.ac_gemm_i8_t.restype = i32
        L.ac_gemm_i8_t.argtypes = [vp, i64, vp, i64, vp, i64, vp, i64, i32, i32, i32, i32, i32, i32, i32, vp]
        L.ac_gemm_i8_planned.restype = i32
        L.ac_gemm_i8_planned.argtypes = L.ac_gemm_i8.argtypes[:-1] + [i32, i32, vp]
        L.ac_gemm_i8_planned_workspace_bytes.restype = sz
        L.ac_gemm_i8_planned_workspace_bytes.argtypes = [i32, i32, i32, i32, i32]
        L.ac_gemm_bf16_ws.restype = i32
        L.ac_gemm_bf16_ws.argtypes = L.ac_gemm_bf16.argtypes[:-1] + [vp, sz, vp]
        L.ac_gemm_bf16_workspace_bytes.restype = sz
        L.ac_gemm_bf16_workspace_bytes.argtypes = [i32, i32, i32]
        L.ac_gemm_bf16_planned.restype = i32
        L.ac_gemm_bf16_planned.argtypes = L.ac_gemm_bf16.argtypes[:-1] + [vp, sz, i32, i32, vp]
        L.ac_gemm_bf16_planned_workspace_bytes.restype = sz
        L.ac_gemm_bf16_planned_workspace_bytes.argtypes = [i32, i32, i32, i32, i32]
        pi32 = ctypes.POINTER(i32)
        L.ac_gemm_i8_auto_plan.restype = None
        L.ac_gemm_i8_auto_plan.argtypes = [i32, i32, i32, i32, pi32, pi32]
        L.ac_gemm_bf16_auto_plan.restype = None
        L.ac_gemm_bf16_auto_plan.argtypes = [i32, i32, i32, pi32, pi32]
        L.ac_status_string.restype = ctypes.c_char_p
        L.ac_status_string.argtypes = [i32]
        L.ac_version.restype = i32
        L.ac_version.argtypes = []
        _lib = L
    return _lib


def native():
    """The compiled side of the functions below (csrc/binding.cpp)."""
    global _native
    if _native is None:
        lib()
        try:
            from . import _binding
        except ImportError as e:
            raise ImportError(f"the compiled binding is missing or does not fit this torch ({e}): build it with "
                              "`python -m paper_2505_18574_amd.build`; there is no fallback path") from e
        _native = _binding
    return _native


def status_string(status: int) -> str:
    return lib().ac_status_string(int(status)).decode()


ac_status_string = status_string


def ac_version() -> int:
    return int(lib().ac_version())


def ac_gemm_i8_workspace_bytes(M: int, N: int, K: int) -> int:
    return int(lib().ac_gemm_i8_workspace_bytes(M, N, K))


def ac_gemm_i8_planned_workspace_bytes(M: int, N: int, K: int, tile: int, splits: int) -> int:
    return int(lib().ac_gemm_i8_planned_workspace_bytes(M, N, K, tile, splits))


def ac_gemm_bf16_workspace_bytes(M: int, N: int, K: int) -> int:
    return int(lib().ac_gemm_bf16_workspace_bytes(M, N, K))


def ac_gemm_bf16_planned_workspace_bytes(M: int, N: int, K: int, tile: int, splits: int) -> int:
    return int(lib().ac_gemm_bf16_planned_workspace_bytes(M, N, K, tile, splits))


def ac_gemm_i8_auto_plan(M: int, N: int, K: int, have_workspace: bool = True):
    """A (tile, splits) of ac_gemm_i8_planned for this shape, to start a search from.  ac_gemm_i8 runs it where no kernel without a code is ahead."""
    tile, splits = ctypes.c_int32(0), ctypes.c_int32(0)
    lib().ac_gemm_i8_auto_plan(M, N, K, int(bool(have_workspace)), ctypes.byref(tile), ctypes.byref(splits))
    return tile.value, splits.value


def ac_gemm_bf16_auto_plan(M: int, N: int, K: int):
    """A (tile, splits) of ac_gemm_bf16_planned for this shape, to start a search from.  ac_gemm_bf16 runs it where no kernel without a code is ahead."""
    tile, splits = ctypes.c_int32(0), ctypes.c_int32(0)
    lib().ac_gemm_bf16_auto_plan(M, N, K, ctypes.byref(tile), ctypes.byref(splits))
    return tile.value, splits.value


# The functions below run once per launch, and on this path a launch takes the GPU no longer than the checks take the
# host.  Each hands its arguments to its compiled namesake first, which takes plain ones (torch.Tensor itself, the right
# types and shapes, ...) and returns a status; a positive one says that something was not plain, and the checks here
# decide whether it is unusual or wrong.
def _ptr(t):
    return None if t is None else t.data_ptr()


def _stream(stream):
    if stream is None:
        return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
    return stream.cuda_stream


def _bad2d(t, dtype, name):
    return ValueError(f"{name}: expected a 2-D row-major device tensor of {dtype}")


def _matrix(t, dtype, name):
    """(rows, columns, row pitch) of a 2-D row-major device tensor of `dtype`."""
    if t.dtype is not dtype or t.ndim != 2 or not t.is_cuda:
        raise _bad2d(t, dtype, name)
    rows, cols = t.shape
    pitch, step = t.stride()
    if cols > 1 and step != 1:
        raise _bad2d(t, dtype, name)
    return rows, cols, pitch


def _ws(workspace):
    if workspace is None:
        return None, 0
    return workspace.data_ptr(), workspace.nbytes


def _bias_i8(bias, M, N):
    """(address, row pitch) of the bias of an M x N output: None, a row of N or an M x N matrix."""
    if bias is None:
        return None, 0
    if bias.dtype is not torch.int32 or not bias.is_cuda:
        raise ValueError("bias: expected int32 device tensor")
    shape = bias.shape
    if len(shape) == 2:
        if tuple(shape) != (M, N) or bias.stride(1) != 1:
            raise ValueError("bias matrix must be M x N row-major")
        return bias.data_ptr(), bias.stride(0)
    if tuple(shape) != (N,) or (N > 1 and bias.stride(0) != 1):
        raise ValueError("bias vector must have N contiguous entries")
    return bias.data_ptr(), 0


def _bias_raw(bias, M, N):
    """(address, row pitch) of the bias of an M x N accumulator: as for _bias_i8, but a vector or a matrix may be larger than
    the output.  What the kernel reads must lie inside it."""
    if bias is None:
        return None, 0
    if bias.dtype != torch.int32 or not bias.is_cuda:
        raise ValueError("bias: expected int32 device tensor")
    if bias.dim() != 2:
        if bias.numel() < N or (N > 1 and not bias.is_contiguous()):
            raise ValueError("bias vector must have N contiguous entries")
        return bias.data_ptr(), 0
    (rows, cols), (pitch, step) = bias.shape, bias.stride()
    # (the library refuses a pitch shorter than a row)
    if not 0 < pitch < N and ((rows < M and pitch != 0) or cols < N or (N > 1 and step != 1)):
        raise ValueError("bias matrix must be M x N row-major")
    return bias.data_ptr(), pitch


def _gemm_i8_args(A, B, bias, C):
    M, K, lda = _matrix(A, torch.int8, "A")
    K2, N, ldb = _matrix(B, torch.int8, "B")
    M2, N2, ldc = _matrix(C, torch.int8, "C")
    if K2 != K or M2 != M or N2 != N:
        raise ValueError("shape mismatch")
    bp, bias_ld = _bias_i8(bias, M, N)
    return A.data_ptr(), lda, B.data_ptr(), ldb, bp, bias_ld, C.data_ptr(), ldc, M, N, K


def ac_gemm_i8(A, B, bias, C, shift: int, act: int = AC_ACT_NONE, workspace=None, stream=None):
    """C[M,N] int8 = stage(A[M,K] . B[K,N] + bias); bias is None, (N,) or (M,N) int32.  Returns C."""
    st = (_native or native()).gemm_i8(A, B, bias, C, shift, act, workspace, stream)
    if st > AC_OK:
        wp, wb = _ws(workspace)
        st = lib().ac_gemm_i8(*_gemm_i8_args(A, B, bias, C), shift, act, wp, wb, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_i8")
    return C


AC_STATIC_SCRATCH_BYTES = 16 << 20


def ac_gemm_i8_static(A, B, bias, C, shift: int, act: int = AC_ACT_NONE, stream=None):
    """ac_gemm_i8 whose K-slice partial sums go through the buffer inside the library (no workspace, no allocation).  Returns C."""
    st = (_lib or lib()).ac_gemm_i8_static(*_gemm_i8_args(A, B, bias, C), shift, act, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_i8_static")
    return C


def ac_gemm_i8_t(A, B, bias, C, shift: int, act: int = AC_ACT_NONE, trans_a: bool = False, trans_b: bool = False, stream=None):
    """ac_gemm_i8 with A given as A^T (K x M) when trans_a and B as B^T (N x K) when trans_b.  Returns C."""
    st = (_native or native()).gemm_i8_t(A, B, bias, C, shift, act, trans_a, trans_b, stream)
    if st > AC_OK:
        M, K, lda = _matrix(A, torch.int8, "A")
        K2, N, ldb = _matrix(B, torch.int8, "B")
        M2, N2, ldc = _matrix(C, torch.int8, "C")
        if trans_a:
            M, K = K, M
        if trans_b:
            K2, N = N, K2
        if K2 != K or M2 != M or N2 != N:
            raise ValueError("shape mismatch")
        bp, bias_ld = _bias_i8(bias, M, N)
        st = lib().ac_gemm_i8_t(A.data_ptr(), lda, B.data_ptr(), ldb, bp, bias_ld, C.data_ptr(), ldc,
                                M, N, K, shift, act, int(bool(trans_a)), int(bool(trans_b)), _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_i8_t")
    return C


def ac_gemm_i8_planned(A, B, bias, C, shift: int, act: int, tile: int, splits: int, workspace=None, stream=None):
    """ac_gemm_i8 with the block tile code (64, 128, 192, 256; 320 / 160 = weight-stationary) and the K split named by the caller.  Returns C."""
    wp, wb = _ws(workspace)
    st = (_lib or lib()).ac_gemm_i8_planned(*_gemm_i8_args(A, B, bias, C), shift, act, wp, wb, tile, splits, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_i8_planned")
    return C


def ac_conv2d_i8(x, w, bias, out, stride: int, pad: int, shift: int, act: int = AC_ACT_NONE, workspace=None, stream=None,
                 plan=None):
    """out[Nb,OH,OW,Cout] int8 = stage(conv(x[Nb,H,W,Cin], w[KH,KW,Cin,Cout]) + bias[Cout]).  Returns out.

    plan = (tile, splits) goes through ac_conv2d_i8_planned."""
    if plan is None:
        st = (_native or native()).conv2d_i8(x, w, bias, out, stride, pad, shift, act, workspace, stream)
        if st == AC_OK:
            return out
        if st < AC_OK:
            raise AcError(st, "ac_conv2d_i8")
    shapes = []
    for t, name in ((x, "x"), (w, "w"), (out, "out")):
        shape = t.shape
        if t.dtype is not torch.int8 or len(shape) != 4 or not t.is_contiguous() or not t.is_cuda:
            raise ValueError(f"{name}: expected a dense 4-D int8 device tensor")
        shapes.append(shape)
    Nb, H, W, Cin = shapes[0]
    KH, KW, Cin2, Cout = shapes[1]
    if Cin2 != Cin:
        raise ValueError("channel mismatch")
    if bias is not None and (bias.dtype is not torch.int32 or tuple(bias.shape) != (Cout,) or not bias.is_contiguous()):
        raise ValueError("bias: expected (Cout,) int32")
    if bias is not None and not bias.is_cuda and not bias.is_pinned():
        raise ValueError("bias: expected int32 device tensor")
    OH = (H + 2 * pad - KH) // stride + 1
    OW = (W + 2 * pad - KW) // stride + 1
    if tuple(shapes[2]) != (Nb, OH, OW, Cout):
        raise ValueError(f"out: expected shape {(Nb, OH, OW, Cout)}")
    wp, wb = _ws(workspace)
    if plan is not None:
        st = (_lib or lib()).ac_conv2d_i8_planned(_ptr(x), _ptr(w), _ptr(bias), _ptr(out), Nb, H, W, Cin, Cout, KH, KW, stride, pad,
                                        shift, act, wp, wb, int(plan[0]), int(plan[1]), _stream(stream))
        if st != AC_OK:
            raise AcError(st, "ac_conv2d_i8_planned")
        return out
    st = (_lib or lib()).ac_conv2d_i8(_ptr(x), _ptr(w), _ptr(bias), _ptr(out), Nb, H, W, Cin, Cout, KH, KW, stride, pad,
                            shift, act, wp, wb, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_conv2d_i8")
    return out


_BF16 = (torch.bfloat16, torch.int16, torch.uint16)


def _gemm_bf16_args(A, B, C):
    dims = []
    for t, name in ((A, "A"), (B, "B")):
        if t.dtype not in _BF16 or t.ndim != 2 or (t.shape[1] > 1 and t.stride(1) != 1) or not t.is_cuda:
            raise ValueError(f"{name}: expected a 2-D row-major bf16 device tensor")
        dims.append((*t.shape, t.stride(0)))
    (M, K, lda), (K2, N, ldb) = dims
    M2, N2, ldc = _matrix(C, torch.float32, "C")
    if K2 != K or M2 != M or N2 != N:
        raise ValueError("shape mismatch")
    return A.data_ptr(), lda, B.data_ptr(), ldb, C.data_ptr(), ldc, M, N, K


def ac_gemm_bf16(A, B, C, alpha: float = 1.0, beta: float = 0.0, stream=None):
    """C[M,N] fp32 = alpha * A[M,K] . B[K,N] + beta * C; A, B are bf16 (torch.bfloat16, or int16/uint16 bit patterns)."""
    st = (_native or native()).gemm_bf16_ws(A, B, C, alpha, beta, None, stream)
    if st > AC_OK:
        st = lib().ac_gemm_bf16(*_gemm_bf16_args(A, B, C), float(alpha), float(beta), _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_bf16")
    return C


def ac_gemm_bf16_ws(A, B, C, alpha: float = 1.0, beta: float = 0.0, workspace=None, stream=None):
    """ac_gemm_bf16 that sums the slices of a cut K range through `workspace` (in a fixed order) when one is given.  Returns C."""
    st = (_native or native()).gemm_bf16_ws(A, B, C, alpha, beta, workspace, stream)
    if st > AC_OK:
        wp, wb = _ws(workspace)
        st = lib().ac_gemm_bf16_ws(*_gemm_bf16_args(A, B, C), float(alpha), float(beta), wp, wb, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_bf16_ws")
    return C


def ac_gemm_bf16_planned(A, B, C, alpha: float, beta: float, tile: int, splits: int, workspace=None, stream=None):
    """ac_gemm_bf16 with the block tile code (64, 128, 192, 256) and the K split named by the caller; a split sums through
    `workspace` when one is given, else with atomic adds into C.  Returns C."""
    wp, wb = _ws(workspace)
    st = (_lib or lib()).ac_gemm_bf16_planned(*_gemm_bf16_args(A, B, C), float(alpha), float(beta), wp, wb, tile, splits, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_bf16_planned")
    return C


def ac_batched_gemm_f32(A, B, C=None, x=None, d=None, y=None, stream=None):
    """Per item: C = A . B (n x n), y = C . x + d.  A, B, C: [batch,n,n]; x, d, y: [batch,n]; fp32 dense."""
    st = (_native or native()).batched_gemm_f32(A, B, C, x, d, y, stream)
    if st == AC_OK:
        return C, y
    if st < AC_OK:
        raise AcError(st, "ac_batched_gemm_f32")
    for t, name in ((A, "A"), (B, "B"), (C, "C"), (x, "x"), (d, "d"), (y, "y")):
        if t is not None and (t.dtype is not torch.float32 or not t.is_contiguous() or not t.is_cuda):
            raise ValueError(f"{name}: expected a dense fp32 device tensor")
    batch, n, n2 = A.shape
    if n != n2 or tuple(B.shape) != (batch, n, n):
        raise ValueError("A, B must be [batch, n, n]")
    if C is not None and tuple(C.shape) != (batch, n, n):
        raise ValueError("C must be [batch, n, n]")
    for t, name in ((x, "x"), (d, "d"), (y, "y")):
        if t is not None and tuple(t.shape) != (batch, n):
            raise ValueError(f"{name} must be [batch, n]")
    st = (_lib or lib()).ac_batched_gemm_f32(_ptr(A), _ptr(B), _ptr(C), _ptr(x), _ptr(d), _ptr(y), n, batch, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_batched_gemm_f32")
    return C, y


def ac_tinympc_forward_f32(Adyn, Bdyn, Kinf, x0, d, u, x_out=None, stream=None):
    """Batched TinyMPC forward pass: u[b,i] = -Kinf x[b,i] - d[b,i]; x[b,i+1] = Adyn x[b,i] + Bdyn u[b,i].

    Adyn [nx,nx], Bdyn [nx,nu], Kinf [nu,nx], x0 [batch,nx], d and u [batch,horizon,nu], x_out [batch,horizon+1,nx] or None."""
    st = (_native or native()).tinympc_forward_f32(Adyn, Bdyn, Kinf, x0, d, u, x_out, stream)
    if st == AC_OK:
        return u, x_out
    if st < AC_OK:
        raise AcError(st, "ac_tinympc_forward_f32")
    for t, name in ((Adyn, "Adyn"), (Bdyn, "Bdyn"), (Kinf, "Kinf"), (x0, "x0"), (d, "d"), (u, "u"), (x_out, "x_out")):
        if t is not None and (t.dtype is not torch.float32 or not t.is_contiguous() or not t.is_cuda):
            raise ValueError(f"{name}: expected a dense fp32 device tensor")
    nx, nu = Bdyn.shape
    batch, horizon, nu2 = d.shape
    if tuple(Adyn.shape) != (nx, nx) or tuple(Kinf.shape) != (nu, nx) or nu2 != nu or tuple(x0.shape) != (batch, nx):
        raise ValueError("shape mismatch")
    if tuple(u.shape) != (batch, horizon, nu) or (x_out is not None and tuple(x_out.shape) != (batch, horizon + 1, nx)):
        raise ValueError("output shape mismatch")
    st = (_lib or lib()).ac_tinympc_forward_f32(_ptr(Adyn), _ptr(Bdyn), _ptr(Kinf), _ptr(x0), _ptr(d), _ptr(u), _ptr(x_out),
                                      nx, nu, horizon, batch, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_tinympc_forward_f32")
    return u, x_out


def ac_gemm_i8_acc32(A, B, bias, C, stream=None):
    """C[M,N] int32 = A[M,K] . B[K,N] + bias (raw accumulator: no scaling, no activation).  Returns C."""
    st = (_native or native()).gemm_i8_acc32(A, B, bias, C, stream)
    if st > AC_OK:
        M, K, lda = _matrix(A, torch.int8, "A")
        K2, N, ldb = _matrix(B, torch.int8, "B")
        M2, N2, ldc = _matrix(C, torch.int32, "C")
        if K2 != K or M2 != M or N2 != N:
            raise ValueError("shape mismatch")
        bp, bias_ld = _bias_raw(bias, M, N)
        st = lib().ac_gemm_i8_acc32(A.data_ptr(), lda, B.data_ptr(), ldb, bp, bias_ld, C.data_ptr(), ldc,
                                    M, N, K, _stream(stream))
    if st != AC_OK:
        raise AcError(st, "ac_gemm_i8_acc32")
    return C
