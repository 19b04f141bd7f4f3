// How far the buffer descriptor of an operand tile reaches, and where a tile begins along the contraction (plain C++, so that a test
// compiles it on the host).
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

// Which starting step a tile of a product takes along the contraction, of as many as there are (modulo these).  Eight neighbouring
// tiles (same column block, neighbouring row blocks) share one, so that their common operand is fetched once into L2.
RMM_RANGE_FN uint32_t start_of_tile(uint32_t tile) { return tile / 8; }
// Y: those that share one are the eight neighbours of 256 x 256 tiles, on tiles of any size, so that its bits are the same on all whose waves do
// not split the contraction.  Smaller tiles take no notice (42 passes and 60 products 1.000 of the time with a start for eight of them, 0.96
// to 1.02).  256 x 256 tiles do where four share one (SORS forward 8192 x 768 -> 1304 1.03, 12000 x 512 -> 1024 1.02 of the time), and
// 128 x 128 tiles of dX with the starts of Y (3000 x 1000 -> 1000, k = 8: backward 27.5 -> 28.5 us), which has its own.
RMM_RANGE_FN uint32_t start_of_place(int64_t m0, int64_t n0, int64_t columns) {
    return (uint32_t)(m0 >> 11) * (uint32_t)((columns + 255) >> 8) + (uint32_t)(n0 >> 8);
}

}  // namespace rmm
