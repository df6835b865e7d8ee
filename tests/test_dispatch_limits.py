"""Dispatch orders at the ends of the range of fo_problem.group_m and num_xcds.

"One band over everything" and "one chiplet per position" may be written as any
large number: the order is the one of a band as tall as the tile grid, for the
plan and for the grids of blocks that the GEMM cuts a plan's output into. The
block grids are evaluated by a program built here from the header that the
kernels are built from.
"""
import ctypes
import os
import subprocess

import pytest

import oracle
import paper_2504_19519_amd as fo

CSRC = os.path.join(os.path.dirname(os.path.abspath(fo.__file__)), "csrc")
INCLUDE = os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include")
LARGE = [1 << 27, 1 << 28, 1 << 29, (1 << 29) + 1, 1 << 30, (1 << 31) - 20, (1 << 31) - 1]

HARNESS = r"""
#include "fo_internal.h"
extern "C" int32_t block_order(int32_t tiles_m, int32_t tiles_n, int32_t tile_m, int32_t tile_n, int32_t block_m,
                               int32_t block_n, int32_t order, int32_t group_m, int32_t num_xcds, int32_t* out) {
    const int32_t rows = (tiles_m * tile_m + block_m - 1) / block_m, cols = (tiles_n * tile_n + block_n - 1) / block_n;
    const int32_t band = fo::block_band(group_m, tile_m, block_m, rows);
    for (int32_t p = 0; p < rows * cols; ++p) out[p] = fo::tile_of_position(p, rows, cols, order, band, num_xcds);
    return band;
}
"""


@pytest.mark.parametrize("order", ["grouped", "xcd"])
@pytest.mark.parametrize("grid", [(4, 4), (4, 1), (4, 2), (1, 3), (7, 5)])
def test_plan_of_large_parameters(grid, order):
    tm, tn = grid
    for group_m, num_xcds in [(g, 8) for g in LARGE] + [(4, x) for x in LARGE] + [(x, x) for x in LARGE]:
        p = fo.plan_groups(64 * tm, 64 * tn, 64, tile_m=64, tile_n=64, order=order, group_m=group_m,
                           num_xcds=num_xcds, num_cus=4, pattern="tile", sizes=[-(-tm * tn // 4)])
        want = oracle.dispatch_order(tm, tn, order, min(group_m, tm), min(num_xcds, tm * tn))
        assert list(p.order) == want == oracle.dispatch_order(tm, tn, order, group_m, num_xcds), (group_m, num_xcds)


@pytest.fixture(scope="module")
def block_order(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fwrapv", "-shared", "-fPIC", "-I", CSRC, "-I", INCLUDE,
                    str(d / "order.cpp"), "-o", str(d / "order.so")], check=True)
    return ctypes.CDLL(str(d / "order.so")).block_order


# tile and block rows and columns: the pairs that the GEMM launches
BLOCKS = [((64, 64), (128, 128)), ((64, 64), (64, 64)), ((64, 64), (64, 32)), ((64, 64), (32, 32)),
          ((256, 128), (128, 128)), ((256, 256), (128, 128))]


@pytest.mark.parametrize("tile,block", BLOCKS)
@pytest.mark.parametrize("order", [1, 2])
def test_every_block_has_one_position(block_order, tile, block, order):
    for tm, tn in [(4, 4), (4, 1), (4, 2), (1, 3), (7, 5)]:
        # (a plan's own band heights are at most its tile rows; the rule for blocks
        # holds for larger ones by itself)
        for group_m in [1, 2, 3, 4, 6, 7] + LARGE:
            for num_xcds in (1, 3, 8):
                rows, cols = -(-tm * tile[0] // block[0]), -(-tn * tile[1] // block[1])
                out = (ctypes.c_int32 * (rows * cols))()
                band = block_order(tm, tn, *tile, *block, order, group_m, num_xcds, out)
                assert band == min(rows, -(-group_m * tile[0] // block[0])), (tm, tn, group_m)
                assert sorted(out) == list(range(rows * cols)), (tm, tn, group_m, num_xcds)
                want = oracle.dispatch_order(rows, cols, "grouped" if order == 1 else "xcd", band, num_xcds)
                assert list(out) == want, (tm, tn, group_m, num_xcds)
