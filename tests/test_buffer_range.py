"""The offsets of weight loads through buffer descriptors (csrc/buffer_range.h), compiled for the host: live
loads read the k-block they name, dead ones (k-blocks past the end of the range, which the pipelines request so
that every stage issues the same number of loads) read zeros whichever way the range check takes a scalar offset
beyond the descriptor's size."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "buffer_range.h"
extern "C" void weight_load(int live, unsigned lane, unsigned scalar, unsigned *out) {
  const deinfer::BufOffsets o = deinfer::weight_load(live != 0, lane, scalar);
  out[0] = o.lane; out[1] = o.scalar;
}
"""


@pytest.fixture(scope="module")
def load(tmp_path_factory):
    d = tmp_path_factory.mktemp("buffer_range")
    (d / "w.cpp").write_text(SRC)
    so = str(d / "w.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2604_17709_amd", "csrc"),
                    "-o", so, str(d / "w.cpp")], check=True)
    fn = ctypes.CDLL(so).weight_load
    fn.argtypes = [ctypes.c_int, ctypes.c_uint, ctypes.c_uint, ctypes.c_void_p]

    def call(live, lane, scalar):
        out = (ctypes.c_uint * 2)()
        fn(int(live), lane, scalar, out)
        return out[0], out[1]
    return call


def in_range_modular(lane, scalar, size):
    """lane < size - scalar in 32-bit unsigned arithmetic."""
    return lane < (size - scalar) % (1 << 32)


def in_range_exact(lane, scalar, size):
    return lane + scalar + 16 <= size


# (a factor of one feature tile: the descriptor ends with the k range; the largest factor below 2^31 bytes)
@pytest.mark.parametrize("tiles,KB", [(1, 1), (1, 2), (1, 7), (3, 1), (3, 33), (1, 2097151), (2097151, 1), (4096, 511)])
def test_dead_weight_loads_read_zeros(load, tiles, KB):
    size = tiles * KB * 1024
    assert size < 1 << 31
    for tile in {0, tiles // 2, tiles - 1}:
        off = tile * KB * 1024
        for kb in list(range(min(KB, 3))) + list(range(max(0, KB - 3), KB + 17)):
            live = kb < KB
            for lane in (0, 16, 1008):                # (the second half of a fragment: 512 bytes on, an offset of the instruction)
                # the tile in the scalar offset (T > 128) or in the lane offset (T <= 128)
                for la, sc in ((lane, off + kb * 1024), (off + lane, kb * 1024)):
                    la, sc = load(live, la, sc)
                    assert in_range_modular(la, sc, size) == live and in_range_exact(la, sc, size) == live
                    if live:
                        assert la + sc == off + kb * 1024 + lane
