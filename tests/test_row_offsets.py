"""Places of rows in memory, on the host.  The 4-bit exact product's tiles: every row of a tile comes from its own row of X, rows past the end from
the last one, however large X is (32-bit offsets from a 64-bit base at the tile).  Right-hand sides in operand tiles: a place
for every element, and room for them.  Tiles of a square, upper half first, and in ranges for the XCDs."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_04453_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("row_offsets")
    (d / "t.cpp").write_text('#include "row_offsets.h"\nextern "C" {\n'
                             'unsigned last_row_offset(int R, int m0, int height, unsigned row_bytes) { return essa_k::last_row_offset(R, m0, height, row_bytes); }\n'
                             'size_t bytes(size_t rows, size_t n) { return essa_k::tiled_rows_bytes(rows, n); }\n'
                             'size_t at(int j, int l, int rows, int n) { return essa_k::tiled_rows_at(j, l, rows, n); }\n'
                             'int width(int nt) { return essa_k::upper_first_width(nt); }\n'
                             'void tile(int x, int y, int nt, int* at) { const essa_k::tile_at t = essa_k::upper_first_tile(x, y, nt); at[0] = t.row; at[1] = t.col; }\n'
                             'int of_xcd(int b, int total) { return essa_k::tile_of_xcd_range(b, total); }\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t.so")], check=True)
    so = ctypes.CDLL(str(d / "t.so"))
    so.last_row_offset.argtypes, so.last_row_offset.restype = [ctypes.c_int] * 3 + [ctypes.c_uint], ctypes.c_uint
    so.bytes.argtypes, so.bytes.restype = [ctypes.c_size_t] * 2, ctypes.c_size_t
    so.at.argtypes, so.at.restype = [ctypes.c_int] * 4, ctypes.c_size_t
    return so


@pytest.mark.parametrize("d_in", [128, 3584, 5120, 8192])
def test_rows_of_a_tile_are_their_own(lib, d_in):
    row_bytes, wrap = 2 * d_in, 2 ** 32 // (2 * d_in)
    for height in (48, 64, 80, 96):
        for R in (257, 300, 1000, wrap - 1, wrap, wrap + 1, wrap + 5, wrap + 100, wrap + 262, 2 * wrap + 50):
            tiles = (R + height - 1) // height
            for t in {0, 1, 2, 3, 4, tiles // 2, tiles - 2, tiles - 1} | {(R - wrap) // height + e for e in (-1, 0, 1)}:
                if not 0 <= t < tiles:
                    continue
                m0 = t * height
                limit = lib.last_row_offset(R, m0, height, row_bytes)
                for row in range(height):
                    off = min(row * row_bytes, limit)
                    assert off < 2 ** 31 and off % row_bytes == 0 and m0 + off // row_bytes == min(m0 + row, R - 1), (d_in, height, R, m0, row)


@pytest.mark.parametrize("rows,n", [(1, 1), (3, 5), (4, 33), (5, 16), (8, 40), (9, 17), (15, 16), (16, 17), (17, 63), (34, 30), (50, 33)])
def test_right_hand_sides_have_places_of_their_own(lib, rows, n):
    n16, height = (n + 15) // 16 * 16, 4 if rows <= 4 else 8 if rows <= 8 else 16
    places = {lib.at(j, l, rows, n) for j in range(rows) for l in range(n16)}
    assert len(places) == rows * n16 and lib.bytes(rows, n) == 4 * n16 * ((rows + height - 1) // height * height) and 4 * max(places) < lib.bytes(rows, n)
    for j in range(rows):                                  # quads are 16 bytes; 16 columns of a tile are in one piece, whatever the row
        tile = j // height * height * n16
        for l in range(0, n16, 4):
            first = tile + l // 16 * height * 16 + (l // 4 % 4 * height + j % height) * 4
            assert [lib.at(j, l + e, rows, n) for e in range(4)] == [first + e for e in range(4)]


def test_right_hand_sides_and_products_fit_three_matrices(lib):
    """An update's scratch beside its products: no more than three matrices in rows took, or than the megabyte that no scratch is smaller than (less what
    else an update keeps there)."""
    for rows in range(3, 1027):
        for n in (1, 17, 100, 120, 241, 400, 895, 3584, 16369, 16384):
            assert lib.bytes(rows, n) + 4 * rows * n <= max(3 * 4 * rows * n, 2 ** 20 - 16384)


def test_right_hand_sides_past_4_gib(lib):
    rows, n = 65536, 16384
    assert lib.bytes(rows, n) == 2 ** 32 and lib.at(rows - 1, n - 1, rows, n) == 2 ** 30 - 1 and lib.at(65520, 0, rows, n) == 65520 * 16384


@pytest.mark.parametrize("nt", [1, 2, 3, 4, 5, 16, 27, 28, 42, 256])
def test_square_has_every_tile_once_and_the_upper_half_first(lib, nt):
    at = (ctypes.c_int * 2)()
    tiles = []
    for y in range(nt):
        for x in range(lib.width(nt)):
            lib.tile(x, y, nt, at)
            if at[0] >= 0:
                tiles.append((at[0], at[1]))
    upper = nt * (nt + 1) // 2
    assert sorted(tiles) == [(i, j) for i in range(nt) for j in range(nt)]
    assert all(i <= j for i, j in tiles[:upper]) and all(i > j for i, j in tiles[upper:])


@pytest.mark.parametrize("total", [1, 5, 7, 8, 9, 15, 16, 196, 252, 505, 1 << 20])
def test_every_xcd_has_a_contiguous_range_of_the_tiles(lib, total):
    ranges = [[lib.of_xcd(b, total) for b in range(xcd, total, 8)] for xcd in range(8)]
    assert [t for r in ranges for t in r] == list(range(total))
