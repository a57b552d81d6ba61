"""The LDS window of the vector-ALU TinyMPC kernel, on the host: for every state and control size and every horizon
around the lengths at which the window's form changes, what the kernel addresses lies inside what the launch reserves."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_18574_amd", "csrc")
SHIM = """
#include "tinympc_window.hpp"
extern "C" void window(int nx, int nu, int horizon, int trajectory, int* out) {
  const ac::TmpcWindow w = ac::tmpc_window(nx, nu, horizon, trajectory != 0);
  const ac::TmpcLayout l = ac::tmpc_layout(nx, nu, horizon, w.chunk, w.whole);
  out[0] = w.whole, out[1] = w.chunk, out[2] = w.floats, out[3] = l.dpitch, out[4] = l.xpitch, out[5] = l.xwin;
}
extern "C" long long pitch(long long steps, int size) { return ac::tmpc_pitch(steps, size); }
"""


@pytest.fixture(scope="module")
def window(tmp_path_factory):
    folder = tmp_path_factory.mktemp("window")
    (folder / "shim.cpp").write_text(SHIM)
    so = str(folder / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", so, str(folder / "shim.cpp")], check=True)
    L = ctypes.CDLL(so)
    L.pitch.restype, L.pitch.argtypes = ctypes.c_longlong, [ctypes.c_longlong, ctypes.c_int]

    def call(nx, nu, horizon, trajectory):
        out = (ctypes.c_int * 6)()
        L.window(nx, nu, horizon, int(trajectory), out)
        return tuple(out)

    call.pitch = L.pitch
    return call


def test_window_holds_what_the_kernel_addresses(window):
    for nx in range(1, 17):
        for nu in range(1, 17):
            for trajectory in (False, True):
                for horizon in list(range(1, 270)) + [1000, 2 ** 31 - 1]:
                    whole, chunk, floats, dpitch, xpitch, xwin = window(nx, nu, horizon, trajectory)
                    where = (nx, nu, horizon, trajectory)
                    assert floats % 4 == 0 and 256 <= floats <= 4096, where  # four such windows are 64 KB
                    assert 1 <= chunk <= horizon and (chunk == horizon or not whole), where
                    # the highest float of problem 15: its last control, its last state
                    steps = horizon if whole else min(chunk, horizon)
                    assert steps * nu <= dpitch and 15 * dpitch + steps * nu <= (xwin if trajectory else floats), where
                    if trajectory:
                        states = (steps + 1 if whole else steps) * nx
                        assert states <= xpitch and xwin + 15 * xpitch + states <= floats, where
                    if not whole:  # a run is divided by one multiply, exact for runs of up to 255 values
                        assert chunk * max(nu, nx if trajectory else 0) <= 255, where


def test_pitch_of_long_horizons(window):
    """Two problems of 2^31 values and more each lie apart by as many."""
    for steps in (5, 2 ** 27, 2 ** 31 - 1, 2 ** 31):
        for size in (1, 3, 16):
            assert window.pitch(steps, size) == steps * size
