"""The rules that give a 16-bit projection to one of the persistent kernels (csrc/gemm_rules.h), compiled for the host."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WRAPPER = r"""
#include "gemm_rules.h"
extern "C" int duo(int M, int N, int K) { return sjd::gemm_duo_applicable(M, N, K); }
extern "C" long long fullest(int M, int N, int rows, int cols) { return sjd::tiles_of_fullest_xcd(M, N, rows, cols); }
"""


def build(tmp_path):
    gxx = shutil.which("g++")
    assert gxx, "g++ is part of the image"
    src = tmp_path / "rules.cpp"
    src.write_text(WRAPPER)
    lib = str(tmp_path / "rules.so")
    subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2505_24791_amd", "csrc"), str(src), "-o", lib], check=True)
    return ctypes.CDLL(lib)


def test_tiles_of_the_fullest_xcd_are_those_that_the_kernels_deal(tmp_path):
    lib = build(tmp_path)
    for rows in (1, 127, 128, 129, 1000, 3000, 4607, 32768):
        for bm in (128, 256):
            panels = -(-rows // bm)
            dealt = [(x + 1) * panels // 8 - x * panels // 8 for x in range(8)]      # as in gemm_p8.hip and gemm_duo.hip
            assert lib.fullest(rows, 3072, bm, 256) == max(dealt) * 12


@pytest.mark.parametrize("N,K", [(1024, 256), (1536, 384), (2048, 512), (2560, 640), (3072, 768), (4096, 1024), (5120, 1280)])
def test_two_workgroups_per_cu_only_where_one_per_cu_needs_a_second_round(tmp_path, N, K):
    """A launch that the 256 x 256 tiles of gemm_p8.hip finish in one round stays there (a pass of width 1024 and 384 tiles: 1141 us
    instead of 1217), unless every CU gets exactly one tile of this kernel."""
    lib = build(tmp_path)
    taken = 0
    for panels in range(1, 400):
        for M in (128 * panels - 127, 128 * panels):
            tiles = panels * N // 256
            one_round = -(-(-(-M // 256)) // 8) * N // 256 <= 32
            one_each = tiles == 256 and -(-panels // 8) * N // 256 <= 32
            assert lib.duo(M, N, K) == (tiles >= 256 and (one_each or not one_round)), M
            taken += lib.duo(M, N, K)
    assert taken > 100


def test_launches_that_the_kernel_does_not_cover(tmp_path):
    lib = build(tmp_path)
    assert lib.duo(32768, 4096, 1024)
    for M, N, K in [(32768, 4096 + 128, 1024), (32768, 4096, 1024 + 64), (32768, 1024, 128), (32768, 1 << 20, 1024), (1, 4096, 1024)]:
        assert not lib.duo(M, N, K), (M, N, K)
