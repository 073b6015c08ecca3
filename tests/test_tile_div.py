"""Divisions of tile and pixel offsets (csrc/tile_div.h), compiled for the host:
exact over the ranges that the kernels use them in."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <algorithm>
#include "tile_div.h"
using namespace onexn;
extern "C" int32_t row(int32_t i, int32_t d) { return row_div(i, d, 1.f / float(d)); }
extern "C" int32_t small(int32_t i, int32_t d) { return small_div(i, 1.f / float(d)); }
// The first divisor in [lo, hi), by steps, of which the last and first two
// offsets of some quotient below `quotients` divide wrongly (0: none).
extern "C" int32_t first_wrong(int64_t lo, int64_t hi, int64_t step, int64_t quotients, bool use_small, int64_t top) {
    for (int64_t d = lo; d < hi; d += step) {
        const float inv = 1.f / float(int32_t(d));
        for (int64_t q = 0; q < quotients; ++q)
            for (int64_t e : {int64_t(0), int64_t(1), d - 1}) {
                const int64_t i = q * d + e;
                if (i >= top || e >= d) continue;
                const int32_t got = use_small ? small_div(int32_t(i), inv) : row_div(int32_t(i), int32_t(d), inv);
                if (got != i / d) return int32_t(d);
            }
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_div")
    src, so = str(d / "div.cpp"), str(d / "div.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                    "-I" + os.path.join(ROOT, "paper_2105_14713_amd", "csrc"), src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.first_wrong.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_bool, ctypes.c_int64]
    return lib


def test_row_div_over_image_sizes(lib):
    """Rows and images of any length (a tile touches up to 257 of them)."""
    top = 2 ** 31 - 4096
    assert lib.first_wrong(1, 2 ** 13, 1, 1024, False, top) == 0
    assert lib.first_wrong(1, 2 ** 24, 1, 3, False, top) == 0
    assert lib.first_wrong(2 ** 13, 2 ** 24, 509, 258, False, top) == 0
    assert lib.first_wrong(2 ** 24, top, 4093, 5, False, top) == 0
    for d in (6556022, 2 ** 22 + 1, 2 ** 30 - 1, 2 ** 30 + 1, top - 1):
        for i in (d - 1, d, min(d + 255, top - 1)):
            assert lib.row(i, d) == i // d


def test_small_div_over_tile_counts(lib):
    assert lib.first_wrong(1, 2 ** 20, 7, 5, True, 2 ** 20) == 0
    assert lib.first_wrong(1, 4096, 1, 256, True, 2 ** 20) == 0
