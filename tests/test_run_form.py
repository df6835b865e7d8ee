"""Which overlapped runs consume their groups together, on the CPU.

The rule is evaluated by a program built here from the header that the library
is built from: by the sizes, and by the limit of the run's waits. A limit that
is enough for each group by itself keeps the launch per group, whose waits are
for one group at a time.
"""
import ctypes
import os
import subprocess

import pytest

import paper_2504_19519_amd as fo

CSRC = os.path.join(os.path.dirname(os.path.abspath(fo.__file__)), "csrc")
INCLUDE = os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")

HARNESS = r"""
#include "fo_internal.h"
extern "C" int together(int64_t M, int64_t N, int64_t K, int32_t W, int sum, int64_t limit_us) {
    fo_plan p;
    p.M = M; p.N = N; p.K = K; p.W = W;
    return fo::consumed_together(p, sum != 0, limit_us);
}
"""


@pytest.fixture(scope="module")
def together(tmp_path_factory):
    d = tmp_path_factory.mktemp("form")
    (d / "form.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-I", INCLUDE, str(d / "form.cpp"),
                    "-o", str(d / "form.so")], check=True)
    f = ctypes.CDLL(str(d / "form.so")).together
    f.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int32, ctypes.c_int, ctypes.c_int64]
    return lambda *a: bool(f(*a))


DEFAULT_US = 2000000


@pytest.mark.parametrize("size,sum_,want", [((256, 256, 256), 1, True), ((1216, 2880, 1984), 1, True),
                                            ((4096, 7168, 2048), 0, True), ((16384, 8192, 2048), 1, True),
                                            ((8192, 8192, 3584), 1, False), ((16384, 4096, 3584), 1, False),
                                            ((8192, 8192, 7168), 1, False)])
def test_by_size(together, size, sum_, want):
    assert together(*size, 256, sum_, DEFAULT_US) == want


@pytest.mark.parametrize("size", [(256, 256, 256), (4096, 7168, 2048), (16384, 8192, 2048)])
@pytest.mark.parametrize("W", [1, 256])
def test_a_short_limit_keeps_a_launch_per_group(together, size, W):
    M, N, K = size
    gemm_us = 2.0 * M * N * K / (W * 5.5e6)
    need = max(10000, 100 * gemm_us)
    short = gemm_us < max(300, 3 * 6.0 * M * N / 5.1e6)
    for limit in (1, 1000, 9999, 10000, int(need) - 1, int(need) + 1, DEFAULT_US, 1 << 62):
        assert together(M, N, K, W, 1, limit) == (short and limit >= need), limit
