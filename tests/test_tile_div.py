"""Divisions of tile and pixel offsets (csrc/tile_div.h), compiled for the host:
exact over the ranges that the kernels use them in."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <initializer_list>
#include "tile_div.h"
using namespace onexn;
extern "C" int32_t div_max() { return kDivMax; }
// The first divisor in [lo, hi) for which an offset near a multiple below `top`
// (and below d + 1024 where `row`) is divided wrongly (0: none).
extern "C" int32_t first_wrong(int64_t lo, int64_t hi, int64_t top, bool row) {
    for (int64_t d = lo; d < hi; ++d) {
        const float inv = 1.f / float(int32_t(d));
        const int64_t end = row ? d + 1024 : top;
        for (int64_t m = 0; m < end; m += d)
            for (int64_t i : {m, m + 1, m + d - 1})
                if (i < end && small_div(int32_t(i), inv) != i / d) return int32_t(d);
        if (row && small_div(int32_t(d + 1023), inv) != (d + 1023) / d) return int32_t(d);
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
    lib.first_wrong.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_bool]
    return lib


def test_row_offsets(lib):
    """Rows and images up to the longest that the kernels divide by, and a tile more."""
    assert lib.first_wrong(1, lib.div_max() + 1, 0, True) == 0


def test_the_limit_is_needed(lib):
    assert lib.first_wrong(1, 1 << 24, 0, True) == 6556022


def test_tile_counts(lib):
    assert lib.first_wrong(1, 4096, 1 << 20, False) == 0
