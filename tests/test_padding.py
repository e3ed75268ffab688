"""Which dwords of the index streams' padding a thread of the encoder clears, on the host: launches have up to 2^32 threads."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_17066_amd", "csrc")
SOURCE = """
#define __host__
#define __device__
#include "vq_padding.hpp"
extern "C" void clear(unsigned char *idx, long long stride, int rows, int from, int count, unsigned block, unsigned block_threads, unsigned thread, unsigned blocks) {
  vq::clear_padding(vq::Padding{idx, stride, rows, from, count}, block, block_threads, thread, blocks);
}
"""


@pytest.fixture(scope="module")
def clear(tmp_path_factory):
    folder = tmp_path_factory.mktemp("padding")
    (folder / "clear.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(folder / "clear.cpp"), "-o", str(folder / "clear.so")])
    f = ctypes.CDLL(str(folder / "clear.so")).clear
    f.argtypes = [ctypes.c_void_p, ctypes.c_longlong] + [ctypes.c_int] * 3 + [ctypes.c_uint] * 4
    return f


@pytest.mark.parametrize("count", [0, 1, 3])
@pytest.mark.parametrize("blocks", [1, 3, (1 << 31) // 256 + 2, (1 << 32) // 256 - 1])
def test_padding_of_any_launch(clear, count, blocks):
    rows, stride, threads = 50, 32, 256
    buffer = np.full((rows + 8, stride), 0xEE, dtype=np.uint8)             # four rows of sentinels on either side
    near = sorted({b for at in (0, (1 << 31) // threads, blocks - 1) for b in range(at - 2, at + 3) if 0 <= b < blocks})
    for block in near:
        for thread in range(threads):
            clear(buffer.ctypes.data + 4 * stride, stride, rows, 5, count, block, threads, thread, blocks)
    want = np.full_like(buffer, 0xEE)
    want[4:-4, 20:20 + 4 * count] = 0
    assert np.array_equal(buffer, want)
