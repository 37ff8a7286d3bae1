"""CPU: what the average reads of a group of 8 parameters that straddles two rows (sdp_avg_group.h, compiled for the host): only rows
that the worker trains, and each parameter of these in its place."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2507_09029_amd import build

SOURCE = '''#include "sdp_avg_group.h"
extern "C" int shift(int split, int first, int second) { return sdp::group_shift(split, first != 0, second != 0); }
extern "C" void align(float* x, int n) { sdp::group_align(*(float (*)[8])x, n); }
'''


@pytest.fixture(scope="module")
def group(tmp_path_factory):
    d = tmp_path_factory.mktemp("group")
    (d / "group.cpp").write_text(SOURCE)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "group.cpp"), "-o", str(d / "group.so")], check=True)
    return ctypes.CDLL(str(d / "group.so"))


@pytest.mark.parametrize("D", [8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 23, 33])
def test_only_rows_that_are_trained_are_read(group, D):
    R = 9
    x = np.arange(1, R * D + 1, dtype=np.float32)
    for off in range(0, R * D - 7, 8):
        row, split = off // D, D - off % D
        if split >= 8:
            continue
        for first, second in ((1, 0), (0, 1), (1, 1)):
            at = off + group.shift(split, first, second)
            trained = [row + i for i, on in enumerate((first, second)) if on]
            assert 0 <= at and at + 8 <= R * D and {(at + i) // D for i in range(8)} <= set(trained), (off, first, second)
            piece = x[at: at + 8].copy()
            group.align(piece.ctypes.data_as(ctypes.c_void_p), at - off)
            want = x[off: off + 8] * np.array([first] * split + [second] * (8 - split), dtype=np.float32)
            assert (piece == want).all(), (off, first, second)
