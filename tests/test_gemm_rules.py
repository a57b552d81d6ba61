"""The launch rules that are arithmetic on sizes, on the host: the shapes of the GPU tests take the kernels they are there for."""
import ctypes
import os
import subprocess

import pytest

import test_gpu_product_tile as product_tile
from paper_2505_18574_amd import ops

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_18574_amd", "csrc")
SHIM = """
#include "gemm_rules.hpp"
extern "C" int product_tile(int M, int N, int K, int st160, int st320) { return ac::choose_product_tile_i8(M, N, K, st160, st320); }
"""
TILE_128X256 = 129


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    folder = tmp_path_factory.mktemp("rules")
    (folder / "shim.cpp").write_text(SHIM)
    so = str(folder / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", so, str(folder / "shim.cpp")], check=True)
    return ctypes.CDLL(so)


def product_tile_of(rules, M, N, K, matrix_bias):
    """The tile of an int8 product on aligned operands whose plan the caller does not name."""
    tiles = -(-M // 64) * -(-N // 64)
    assert tiles > 512 or (tiles > 256 and K < 4096)
    assert ops.ac_gemm_i8_auto_plan(M, N, K, False)[0] != 32
    return rules.product_tile(M, N, K, *(1 <= K <= limit and not matrix_bias for limit in (2048, 1536)))


def test_product_tile_shapes(rules):
    for matrix in (False, True):
        for shape in product_tile.TILE_128X256:
            assert product_tile_of(rules, *shape, matrix) == TILE_128X256, shape
        for M, N, K in product_tile.SEVERAL_TO_A_WORKGROUP:
            assert product_tile_of(rules, M, N, K, matrix) == TILE_128X256 and -(-M // 128) * -(-N // 256) > 512, (M, N, K)
    assert [product_tile_of(rules, *shape, False) for shape in product_tile.OTHER_CODES] == [320, 128]
