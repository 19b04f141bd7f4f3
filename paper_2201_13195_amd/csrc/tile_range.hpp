// How far the buffer descriptor of an operand tile reaches (plain C++, so that a test compiles it on the host).
#pragma once
#include <stdint.h>

#ifdef __HIP__
#define RMM_RANGE_FN __host__ __device__ constexpr
#else
#define RMM_RANGE_FN constexpr
#endif

namespace rmm {

// Bytes from the descriptor's base to the end of the dword that holds the last valid element of a tile.
//   ES         bytes of an element (2 or 4)
//   KROWS      rows run along the contraction
//   rows_left  rows (KROWS) or columns from the tile's first to the operand's last; at most `tile_rows` are the tile's
//   left       contraction elements of the tile that exist; with none the range is empty
//   skew       elements between the base, which is on a dword, and the first element (0 or 1, bf16 only)
// The descriptor's range ends inside the operand's last dword, whose other half, if any, lies on the same
// page: nothing beyond it is ever touched, wherever the operand ends.
// `I`: 32 bits hold the range of a tile of 128 rows of fewer than 2^22 elements (2^31 bytes, with no sign); on the device they are a
// few scalar instructions where 64 are compared in vector ones.
template <int ES, bool KROWS, typename I>
RMM_RANGE_FN I tile_range_bytes(I rows_left, I tile_rows, I ld, I left, I skew) {
    if (left <= 0) return 0;
    const I rows = rows_left < tile_rows ? rows_left : tile_rows;
    const I elems = KROWS ? (rows - 1) * ld + left : (left - 1) * ld + rows_left;
    return (((elems + skew) * ES) + 3) & ~(I)3;
}

}  // namespace rmm
