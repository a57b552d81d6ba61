"""The compiled binding takes plain arguments and leaves everything else to the checks of ops.py."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2505_18574_amd import ops

PYTHON = 1


def i8(*s):
    return torch.zeros(s, dtype=torch.int8)


def f32(*s):
    return torch.zeros(s)


def test_what_is_not_plain_is_left_to_python():
    n = ops.native()
    A, C, b = i8(4, 4), i8(4, 4), torch.zeros(4, dtype=torch.int32)
    for args in ((A, A, b, C, 1, 0, None, None), (None,) * 8, ("A",) * 8, (A, A, b, C, 1.5, 0, None, None), (A,), (A,) * 9):
        assert n.gemm_i8(*args) == PYTHON  # tensors on the host, no tensors, other counts
    assert n.gemm_i8_t(A, A, b, C, 1, 0, False, 1, None) == PYTHON
    assert n.gemm_i8_acc32(A, A, b, C, None) == PYTHON
    assert n.conv2d_i8(i8(1, 4, 4, 2), i8(3, 3, 2, 4), None, i8(1, 4, 4, 4), 1, 1, 1, 0, None, None) == PYTHON
    assert n.gemm_bf16_ws(A, A, C, 1.0, 0.0, None, None) == PYTHON
    assert n.batched_gemm_f32(f32(2, 3, 3), f32(2, 3, 3), None, None, None, None, None) == PYTHON
    assert n.tinympc_forward_f32(*[f32(2, 2)] * 7, None) == PYTHON


def test_errors_are_those_of_the_python_checks():
    A, C = i8(4, 4), i8(4, 4)
    with pytest.raises(ValueError, match="A: expected a 2-D row-major device tensor"):
        ops.ac_gemm_i8(A, A, None, C, 1)
    with pytest.raises(ValueError, match="A: expected a 2-D row-major bf16 device tensor"):
        ops.ac_gemm_bf16_ws(A, A, C)
    with pytest.raises(ValueError, match="x: expected a dense 4-D int8 device tensor"):
        ops.ac_conv2d_i8(A, A, None, C, 1, 0, 1)
    with pytest.raises(ValueError, match="A: expected a dense fp32 device tensor"):
        ops.ac_batched_gemm_f32(f32(1, 2, 2), f32(1, 2, 2), f32(1, 2, 2))
    with pytest.raises(AttributeError):
        ops.ac_gemm_i8(None, A, None, C, 1)


class OnDevice(torch.Tensor):
    """A host tensor that says it is on the device, for the checks of ops.py."""
    is_cuda = property(lambda self: True)


class Pinned(torch.Tensor):
    is_pinned = lambda self: True


class Launches:
    """A library that notes what would have been launched."""

    def __init__(self, monkeypatch):
        self.calls = []
        monkeypatch.setattr(ops, "lib", lambda: self)
        monkeypatch.setattr(ops, "_lib", self)

    def __getattr__(self, name):
        return lambda *args: self.calls.append((name, args)) or ops.AC_OK


class NullStream:
    cuda_stream = 0


def test_raw_accumulator_refuses_a_bias_it_would_read_beyond(monkeypatch):
    """What the kernel reads (row m at data + m * pitch, N values in a row) lies inside the bias, and is what it holds."""
    ops.native()
    lib = Launches(monkeypatch)
    A, B, C = (i8(5, 8).as_subclass(OnDevice), i8(8, 6).as_subclass(OnDevice), torch.zeros((5, 6), dtype=torch.int32).as_subclass(OnDevice))
    i32 = lambda *s: torch.zeros(s, dtype=torch.int32)
    call = lambda b: ops.ac_gemm_i8_acc32(A, B, b.as_subclass(OnDevice), C, stream=NullStream)
    for bad in (i32(5), i32(0), i32(1, 6), i32(4, 6), i32(5, 9)[:, :5], i32(12)[::2], i32(5, 12)[:, ::2], i32(1, 1, 5)):
        with pytest.raises(ValueError, match="bias"):
            call(bad)
    assert lib.calls == []
    pitches = []
    for good in (i32(6), i32(9), i32(5, 6), i32(7, 9), i32(5, 9)[:, 2:8], i32(6).expand(5, 6), i32(1, 1, 6)):
        call(good)
        name, args = lib.calls.pop()
        assert name == "ac_gemm_i8_acc32" and args[4] == good.data_ptr()
        pitches.append(args[5])
    assert pitches == [0, 0, 6, 9, 9, 0, 0]
    A, B, C = i8(5, 8).as_subclass(OnDevice), i8(8, 1).as_subclass(OnDevice), torch.zeros((5, 1), dtype=torch.int32).as_subclass(OnDevice)
    for good, pitch in ((i32(2)[::2], 0), (i32(5, 1), 1), (i32(5, 3)[:, 1:2], 3), (i32(1, 5).t(), 1)):  # one column: rows of one value
        call(good)
        assert lib.calls.pop()[1][5] == pitch


def test_convolution_refuses_a_bias_in_pageable_host_memory(monkeypatch):
    ops.native()
    lib = Launches(monkeypatch)
    x, w, out = (i8(*s).as_subclass(OnDevice) for s in ((1, 4, 4, 2), (3, 3, 2, 4), (1, 4, 4, 4)))
    bias = torch.zeros(4, dtype=torch.int32)
    for plan in (None, (64, 1)):
        with pytest.raises(ValueError, match="bias"):
            ops.ac_conv2d_i8(x, w, bias, out, 1, 1, 1, stream=NullStream, plan=plan)
        assert lib.calls == []
        for there in (bias.as_subclass(OnDevice), bias.as_subclass(Pinned)):  # the GPU reads pinned memory
            ops.ac_conv2d_i8(x, w, there, out, 1, 1, 1, stream=NullStream, plan=plan)
            assert lib.calls.pop()[1][2] == bias.data_ptr()


def test_a_copied_package_loads_its_own_library(tmp_path):
    """One library in the process, the one beside the binding: not also that of the tree it was built in."""
    here = os.path.dirname(ops.LIB_PATH)
    copy = tmp_path / os.path.basename(here)
    copy.mkdir()
    for name in os.listdir(here):
        if name.endswith((".py", ".so")):
            shutil.copy(os.path.join(here, name), copy)
    code = f"from {copy.name} import ops; ops.native(); print(*{{l.split()[-1] for l in open('/proc/self/maps') if 'libac_mi355x' in l}})"
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True,
                       env={**os.environ, "PYTHONPATH": str(tmp_path), "LD_LIBRARY_PATH": here + ":" + os.environ.get("LD_LIBRARY_PATH", "")})
    assert r.returncode == 0, r.stderr
    assert r.stdout.split() == [str(copy / os.path.basename(ops.LIB_PATH))]


class Sub(torch.Tensor):
    pass


@pytest.mark.gpu
def test_plain_and_unusual_arguments_give_the_same_result():
    g = np.random.default_rng(3)
    A, B = (torch.from_numpy(g.integers(-128, 128, s).astype(np.int8)).cuda() for s in ((40, 64), (64, 48)))
    bias = torch.arange(48, dtype=torch.int32, device="cuda") * 300
    new = lambda: torch.full((40, 48), 5, dtype=torch.int8, device="cuda")
    n = ops.native()
    C = new()
    assert n.gemm_i8(A, B, bias, C, 9, 1, None, None) == ops.AC_OK
    assert n.gemm_i8(A, B, bias, C, 99, 1, None, None) == ops.AC_ERR_SHIFT
    assert n.gemm_i8(A, B.t(), bias, C, 9, 1, None, None) == PYTHON      # not row-major
    assert n.gemm_i8(A, B, bias[:-1], C, 9, 1, None, None) == PYTHON     # a bias of another length
    with pytest.raises(ops.AcError) as e:
        ops.ac_gemm_i8(A, B, bias, C, 99)
    assert e.value.status == ops.AC_ERR_SHIFT
    with pytest.raises(ValueError, match="bias vector"):
        ops.ac_gemm_i8(A, B, bias[:-1], C, 9)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    D, E, F = new(), new(), new()
    with torch.cuda.stream(side):
        ops.ac_gemm_i8(A, B, bias, D, np.int64(9), np.int32(1))            # integers of numpy
    ops.ac_gemm_i8(A, B, bias, E, 9, act=1, stream=side)                   # a stream by name
    side.synchronize()
    ops.ac_gemm_i8(A.as_subclass(Sub), B, bias.expand(40, 48).contiguous(), F, True + 8, True)  # a subclass, a bias matrix, bools
    for out in (D, E, F):
        assert torch.equal(out, C)
    P, Q = torch.randn(33, 16, device="cuda").bfloat16(), torch.randn(16, 24, device="cuda").bfloat16()
    R, S = torch.zeros(33, 24, device="cuda"), torch.zeros(33, 24, device="cuda")
    ops.ac_gemm_bf16(P, Q, R)
    ops.ac_gemm_bf16(P.view(torch.int16), Q.view(torch.uint16), S, 1, 0)   # bit patterns, integer factors
    assert torch.equal(R, S)
