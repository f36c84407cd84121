import ctypes
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def orc32():
    from oracle import Oracle
    return Oracle("f32")


@pytest.fixture(scope="session")
def orc64():
    from oracle import Oracle
    return Oracle("f64")


LAUNCH_RULES = r"""
#include "gemm_rules.h"
#include "seq_groups.h"
extern "C" {
int duo(int M, int N, int K) { return sjd::gemm_duo_applicable(M, N, K); }
int dma_before_ring(int M, int N, int gelu) { return sjd::gemm_dma_before_ring(M, N, gelu != 0); }
long long fullest(int M, int N, int rows, int cols) { return sjd::tiles_of_fullest_xcd(M, N, rows, cols); }
int xcds_per_group(int W, int batch) { return sjd::seq_xcds_per_group(W, batch); }
int xcds_per_group_on(int W, int batch, int n_cus) { return sjd::seq_xcds_per_group(W, batch, n_cus); }
int rows_ahead(int B, int heads, int width, int T, int n_cus, int xpg) { return sjd::seq_rows_ahead(B, heads, width, T, n_cus, xpg); }
}
"""


@pytest.fixture(scope="session")
def launch_rules(tmp_path_factory):
    """The rules by which the library picks a kernel (plain C++ headers beside the kernels), compiled for the host."""
    gxx = shutil.which("g++")
    assert gxx, "g++ is part of the image"
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", str(d / "rules.so")
    src.write_text(LAUNCH_RULES)
    subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2505_24791_amd", "csrc"), str(src), "-o", lib], check=True)
    return ctypes.CDLL(lib)
