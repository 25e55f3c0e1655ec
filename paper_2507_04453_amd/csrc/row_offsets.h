// Places of rows in memory and of tiles in a matrix: plain constexpr C++, so that a test can run on the host what the kernels run.
#pragma once
#include <cstddef>
#include <cstdint>

namespace essa_k {

// Loads whose 64-bit base is row m0 reach row `row` of a tile of `height` rows at min(row * row_bytes, last_row_offset): rows past the
// last one read that one.  The rows are bounded by the tile before they are multiplied: what is left of X behind m0 can be more than 4 GB.
constexpr uint32_t last_row_offset(int R, int m0, int height, uint32_t row_bytes) {
    const int left = R - 1 - m0;
    return (uint32_t)(left < height - 1 ? left : height - 1) * row_bytes;
}

// Right-hand sides of the product with the basis (a matrix of `rows` rows and n columns of floats) lie in operand tiles of 16 rows (8 or 4 where there
// are no more) and 16 columns, tile (j / 16, l / 16), inside it [l / 4 % 4][row][l % 4] -- a wave's load is one contiguous kilobyte.  Columns
// past n are zero, rows past the last one anything finite or not: they are not read.  With their products they take no more than three
// matrices in rows, which a scratch that cannot grow may have been made for, or than the megabyte that no scratch is smaller than.
constexpr int tiled_rows_shift(int rows) { return rows <= 4 ? 2 : rows <= 8 ? 3 : 4; }
constexpr size_t tiled_rows_bytes(size_t rows, size_t n) {
    const int s = tiled_rows_shift(rows < 16 ? (int)rows : 16);
    return (((rows + (1 << s) - 1) >> s) * ((n + 15) / 16)) << (s + 6);
}
constexpr size_t tiled_rows_at(int j, int l, int rows, int n) {      // the float of row j, column l
    const int s = tiled_rows_shift(rows);
    return (((((size_t)(j >> s) * ((n + 15) >> 4) + (l >> 4)) * 4 + (l >> 2 & 3)) << s) + (j & ((1 << s) - 1))) * 4 + (l & 3);
}

// The tiles of a square of nt x nt for workgroups of a grid of upper_first_width(nt) x nt: the nt (nt + 1) / 2 tiles on and above the diagonal come first (row by row,
// the last row in what the first one leaves free, the last but one in the second's and so on), then the ones below; the last two of a line have none there with nt even.
struct tile_at { int row, col; };
constexpr int upper_first_width(int nt) { return nt + 1 - (nt & 1); }
constexpr tile_at upper_tile(int x, int y, int nt) {
    const int odd = nt & 1;
    return x + odd > y ? tile_at{y, x - 1 + odd} : tile_at{nt - 1 + odd - y, nt - 1 - x};
}
constexpr tile_at upper_first_tile(int x, int y, int nt) {          // row < 0: none
    const int lines = (nt + 1) / 2;
    if (y < lines) return upper_tile(x, y, nt);
    if (x >= upper_first_width(nt - 1)) return tile_at{-1, -1};
    const tile_at mirror = upper_tile(x, y - lines, nt - 1);
    return tile_at{mirror.col + 1, mirror.row};
}

// Workgroups go round-robin over the 8 XCDs: the tile that workgroup b of `total` takes so that every XCD has a contiguous range of them (the first total % 8
// XCDs one more than the others).
constexpr int tile_of_xcd_range(int b, int total) {
    const int xcd = b & 7, more = total & 7;
    return xcd * (total >> 3) + (xcd < more ? xcd : more) + (b >> 3);
}

}  // namespace essa_k
