"""CPU: which form of the bf16 attention core a call takes (sdp_attn_rule.h, compiled for the host)."""
import ctypes
import os
import subprocess

import pytest

from paper_2507_09029_amd import build

SOURCE = '''#include "sdp_attn_rule.h"
extern "C" int waves(int hd, int64_t S, int64_t pairs) { return sdp::core_waves(hd, S, pairs); }
extern "C" int merged(int hd, int64_t S, int64_t pairs) { return sdp::core_merged_backward(hd, S, pairs); }
'''


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(SOURCE)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "rule.cpp"), "-o", str(d / "rule.so")], check=True)
    lib = ctypes.CDLL(str(d / "rule.so"))
    for f in (lib.waves, lib.merged):
        f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64]
    return lib


@pytest.mark.parametrize("hd", [72, 96, 128])
def test_eight_waves_share_a_walk(rule, hd):
    # 512 tokens on and up to 8 pairs, whether or not the tokens are a multiple of 32
    assert [rule.waves(hd, S, n) for S, n in ((511, 4), (512, 4), (513, 8), (2047, 8), (2048, 8), (2048, 9))] == [4, 8, 8, 8, 8, 4]
    # and while one wave along the walked axis has at most 336 workgroups: 256, 336 | 344, 512
    assert [rule.waves(hd, S, n) for S, n in ((4096, 8), (5376, 8), (5377, 8), (8192, 8))] == [8, 8, 1, 1]
    assert [rule.waves(hd, S, n) for S, n in ((8192, 2), (8192, 4), (21504, 2), (21505, 2), (1 << 17, 1), (1 << 17, 8))] == [8, 8, 8, 1, 1, 1]


def test_other_heads_never_take_eight(rule):
    assert [rule.waves(64, S, n) for S, n in ((2048, 8), (4096, 8), (4096, 9))] == [4, 4, 1]
    assert [rule.waves(128, 256, n) for n in (96, 97)] == [4, 1]


def test_one_backward_launch_only_where_the_walk_is_split(rule):
    for hd in (64, 72, 128):
        for S in (1, 31, 32, 33, 128, 200, 511, 512, 1024, 1025, 1056, 2048, 5376, 8192, 65536):
            for n in (1, 2, 7, 8, 9, 28, 56, 57, 192, 193, 224, 225, 256, 257):
                assert not rule.merged(hd, S, n) or rule.waves(hd, S, n) > 1, (hd, S, n)
    assert [rule.merged(hd, S, n) for hd, S, n in ((128, 1024, 8), (128, 1025, 8), (128, 224, 32), (128, 224, 33), (64, 32, 256), (64, 32, 257), (128, 32, 193))] \
        == [1, 0, 1, 0, 1, 0, 0]


def test_one_backward_launch_of_narrow_heads_while_its_reads_are_few(rule):
    # up to 384 blocks of 32 rows; beyond, blocks x tokens up to 2^20
    assert [rule.merged(64, S, n) for S, n in ((2048, 8), (12288, 1), (4096, 3), (1024, 24), (1024, 32), (511, 64))] == [1, 1, 1, 1, 1, 1]
    assert [rule.merged(64, S, n) for S, n in ((2048, 9), (2112, 8), (3000, 7), (4096, 4), (6000, 5), (8192, 4), (12320, 1))] == [0, 0, 0, 0, 0, 0, 0]
