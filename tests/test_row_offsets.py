"""Row offsets of the 4-bit exact product's tiles, on the host: every row of a tile comes from its own row of X, rows past the end from the last
one, however large X is (32-bit offsets from a 64-bit base at the tile)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_04453_amd", "csrc")


@pytest.fixture(scope="module")
def last_row_offset(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_offsets")
    (d / "t.cpp").write_text('#include "row_offsets.h"\nextern "C" unsigned f(int R, int m0, int height, unsigned row_bytes) {\n'
                             '    return essa_k::last_row_offset(R, m0, height, row_bytes);\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    f = ctypes.CDLL(str(d / "t.so")).f
    f.argtypes, f.restype = [ctypes.c_int] * 3 + [ctypes.c_uint], ctypes.c_uint
    return f


@pytest.mark.parametrize("d_in", [128, 3584, 5120, 8192])
def test_rows_of_a_tile_are_their_own(last_row_offset, d_in):
    row_bytes, wrap = 2 * d_in, 2 ** 32 // (2 * d_in)
    for height in (48, 64, 80, 96):
        for R in (257, 300, 1000, wrap - 1, wrap, wrap + 1, wrap + 5, wrap + 100, wrap + 262, 2 * wrap + 50):
            tiles = (R + height - 1) // height
            for t in {0, 1, 2, 3, 4, tiles // 2, tiles - 2, tiles - 1} | {(R - wrap) // height + e for e in (-1, 0, 1)}:
                if not 0 <= t < tiles:
                    continue
                m0 = t * height
                limit = last_row_offset(R, m0, height, row_bytes)
                for row in range(height):
                    off = min(row * row_bytes, limit)
                    assert off < 2 ** 31 and off % row_bytes == 0 and m0 + off // row_bytes == min(m0 + row, R - 1), (d_in, height, R, m0, row)
