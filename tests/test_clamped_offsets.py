"""The offsets at which the next layer's epilogue reads the (unpadded) magnitude sums, compiled for the host from
the kernels' own header: inside the array for every element of every tile, whole tiles of 256 x 256 included."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2311_05782_amd import build


@pytest.fixture(scope="module")
def offset(tmp_path_factory):
    d = tmp_path_factory.mktemp("clamped")
    src, lib = str(d / "host.cpp"), str(d / "host.so")
    with open(src, "w") as f:
        f.write('#include "clamped.hpp"\n'
                'extern "C" uint32_t offset(int row, int col, int M, int N) { return fi::clamped_word_offset(row, col, M, N); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    "-I", build.CSRC, src, "-o", lib], check=True)
    fn = C.CDLL(lib).offset
    fn.restype, fn.argtypes = C.c_uint32, [C.c_int] * 4
    return fn


@pytest.mark.parametrize("M,N", [(1, 1), (1, 1 << 20), (3, 5), (33, 257), (257, 4096), (255, 4), (256, 256), (63, (1 << 24) + 1)])
def test_no_element_of_a_tile_is_read_outside_the_array(offset, M, N):
    rows = range((M + 255) // 256 * 256)
    end = (N + 255) // 256 * 256
    cols = sorted({c for x in (0, N, end) for c in range(x - 3, x + 3) if 0 <= c < end} | {N // 2})
    for row in rows:
        for col in cols:
            at = offset(row, col, M, N)
            assert at % 4 == 0 and at + 4 <= M * N * 4, (row, col)
            if row < M and col < N:
                assert at == (row * N + col) * 4
