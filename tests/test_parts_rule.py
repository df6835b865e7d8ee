"""Which unsignalled GEMMs of larger tiles run in 128x128 blocks, on the CPU.

The rule is evaluated by a program built here from the header that the library is
built from, at the sizes where tiles and blocks were measured against each other
(the faster form is expected; sizes within 3 % are left out): with blocks in
pairs on a compute unit, and where reserved units keep them single.
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
extern "C" int parts(int tile_n, int64_t tiles, int64_t W, int64_t K, int share_cus) {
    return fo::takes_parts(tile_n, tiles, W, K, share_cus != 0);
}
"""


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    (d / "parts.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, "-I", INCLUDE, str(d / "parts.cpp"),
                    "-o", str(d / "parts.so")], check=True)
    f = ctypes.CDLL(str(d / "parts.so")).parts
    f.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int]
    return lambda *a: bool(f(*a))


# tile_n, tiles, K, us in tiles, us in blocks
RESERVED = [(128, 120, 256, 9.4, 8.0), (128, 120, 4096, 53, 34), (128, 128, 256, 9.5, 11.7),
            (128, 240, 1024, 20.4, 22.2), (128, 240, 4096, 62, 65), (128, 300, 1024, 33.8, 29.6),
            (128, 300, 4096, 106, 89), (128, 360, 4096, 109, 96), (128, 480, 1024, 38.3, 41),
            (256, 60, 1024, 25, 12.6), (256, 60, 4096, 72, 34), (256, 120, 256, 13.5, 12.4), (256, 120, 4096, 75, 65),
            (256, 250, 4096, 161, 145), (256, 300, 4096, 163, 156), (256, 320, 1024, 51.2, 54.2)]
SHARED = [(128, 128, 4096, 52, 32), (128, 192, 4096, 55, 48), (128, 256, 1024, 20, 18), (128, 320, 4096, 107, 85),
          (128, 512, 1024, 37, 34), (256, 64, 4096, 72, 33), (256, 128, 4096, 74, 57), (256, 192, 4096, 82, 90),
          (256, 256, 4096, 101, 119), (256, 320, 4096, 168, 158), (256, 384, 1024, 55, 51), (256, 448, 4096, 190, 214)]


@pytest.mark.parametrize("share,W,rows", [(False, 240, RESERVED), (True, 256, SHARED)], ids=["single", "pairs"])
def test_the_faster_form(parts, share, W, rows):
    for tile_n, tiles, K, in_tiles, in_blocks in rows:
        assert parts(tile_n, tiles, W, K, share) == (in_blocks < in_tiles), (tile_n, tiles, K)


@pytest.mark.parametrize("tile_n", [128, 256])
def test_many_tiles_stay_whole(parts, tile_n):
    for share in (False, True):
        for W in (1, 7, 240, 256):
            for tiles in (2 * W + 1, 3 * W, 4 * W + 1, 1000 * W):
                if tiles > 2 * W:
                    assert not parts(tile_n, tiles, W, 4096, share), (share, W, tiles)
