"""Host build of the launch geometry of the fp32 attention kernels: layers of
more blocks than one launch can hold (2^32 threads) go out in several launches
that cover every block once, all others in one.  Runs on the CPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HDR_DIR = os.path.join(ROOT, "paper_2505_00315_amd", "csrc")

SRC = r"""
#include "launch_parts.h"
extern "C" int t_waves(int n) { return mosa::f32_attn_waves(n, 8); }
extern "C" int t_parts(uint64_t blocks, uint32_t threads, uint64_t* out, int cap, int stop) {
    int k = 0;
    const int e = mosa::launch_parts(blocks, threads, [&](uint32_t first, uint32_t count) {
        if (k < cap) out[2 * k] = first, out[2 * k + 1] = count;
        return ++k == stop ? -1 : 0;
    });
    return e ? -k : k;
}
"""


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_parts")
    (d / "t.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", HDR_DIR,
                           str(d / "t.cpp"), "-o", str(d / "t.so")])
    return ctypes.CDLL(str(d / "t.so"))


def _plan(lib, blocks, threads, stop=0):
    out = np.zeros((64, 2), np.uint64)
    k = lib.t_parts(ctypes.c_uint64(blocks), ctypes.c_uint32(threads), out.ctypes.data_as(ctypes.c_void_p), 64, stop)
    return k, [(int(a), int(b)) for a, b in out[: abs(k)]]


# (b, h) pairs and rows: the sizes at which the backward (twice the blocks) and
# the forward pass 2^32 threads, one block short of that, the most rows of any
# layer (2e9, in groups of 1 row and of 128), and ordinary ones
@pytest.mark.parametrize("bh,n", [(16383 * 5, 1024), (8193 * 64, 113), (8192 * 64 - 1, 113), (2000000000, 1),
                                  (15625000, 128), (32, 512), (1, 1)])
@pytest.mark.parametrize("passes", [1, 2])
def test_every_block_once_within_the_limit(parts, bh, n, passes):
    threads = 64 * parts.t_waves(n)
    blocks = passes * bh * ((n + 15) // 16)
    k, p = _plan(parts, blocks, threads)
    assert k == len(p) == -(-blocks // (0xffffffff // threads))
    at = 0
    for first, count in p:
        assert first == at and 0 < count and count * threads < 1 << 32
        at += count
    assert at == blocks
    if blocks * threads < 1 << 32:
        assert k == 1


def test_stops_at_a_failed_launch(parts):
    k, p = _plan(parts, 3 << 24, 512, stop=2)
    assert k == -2 and len(p) == 2
    assert _plan(parts, 0, 512) == (0, [])


@pytest.mark.parametrize("n,waves", [(1, 1), (16, 1), (17, 2), (33, 2), (49, 4), (97, 4),
                                     (113, 8), (16384, 8)])
def test_waves(parts, n, waves):
    assert parts.t_waves(n) == waves
