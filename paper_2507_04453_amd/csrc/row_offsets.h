// Byte offsets of a tile's rows: plain constexpr C++, so that a test can run on the host what the kernels run.
#pragma once
#include <cstdint>

namespace essa_k {

// Loads whose 64-bit base is row m0 reach row `row` of a tile of `height` rows at min(row * row_bytes, last_row_offset): rows past the
// last one read that one.  The rows are bounded by the tile before they are multiplied: what is left of X behind m0 can be more than 4 GB.
constexpr uint32_t last_row_offset(int R, int m0, int height, uint32_t row_bytes) {
    const int left = R - 1 - m0;
    return (uint32_t)(left < height - 1 ? left : height - 1) * row_bytes;
}

}  // namespace essa_k
