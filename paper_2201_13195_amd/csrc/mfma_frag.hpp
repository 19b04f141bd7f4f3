// Operand fragments of v_mfma_f32_32x32x16_bf16 and the LDS layouts they are read from, shared by
// the bf16 kernels (mfma_kernels.hpp) and the fp32 ones (plain_kernels.hpp).
#pragma once
#include "common.hpp"

namespace rmm {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// K-contiguous LDS tiles are not padded: row r keeps its 16-byte chunk c at chunk position
// c ^ ((r / (16 / U)) % U), U = chunks per row.  Then the 16 lanes that the LDS serves together hit
// 16 different 16-byte bank groups both when a tile is written (consecutive lanes = consecutive
// chunks of U-chunk rows) and when fragments are read (consecutive lanes = consecutive rows, same
// chunk); a padded layout can only make one of the two conflict-free.
template <int BK>
__device__ __forceinline__ int kchunk_pos(int row, int chunk) {
    constexpr int U = BK / 8, G = 16 / U;
    static_assert(U == 4 || U == 8 || U == 16, "BK of 32, 64 or 128");
    return chunk ^ ((row / G) % U);
}
constexpr int TPAD = 32;  // elements of padding per row of a transposed-read LDS tile (row stride = 64 mod 256 B)

// Operand fragment of the 32x32x16 MFMA from a K-contiguous LDS tile (rows of BK elements,
// chunks placed by kchunk_pos): lane l holds row (l % 32), contraction elements 8*(l / 32) .. +7.
template <int BK>
__device__ __forceinline__ int kcontig_offset(int row0, int kk0, int lane) {  // elements
    const int row = row0 + (lane & 31), chunk = (kk0 >> 3) + (lane >> 5);
    return row * BK + kchunk_pos<BK>(row, chunk) * 8;
}
template <int BK>
__device__ __forceinline__ bf16x8_t frag_kcontig(const bf16_t *tile, int row0, int kk0, int lane) {
    const int row = row0 + (lane & 31), chunk = (kk0 >> 3) + (lane >> 5);
    return *reinterpret_cast<const bf16x8_t *>(tile + row * BK + kchunk_pos<BK>(row, chunk) * 8);
}

// Same fragment from a tile stored [contraction row][column]: two transposing
// reads.  Within a block of 16 lanes, lane i points at row (i / 4), columns
// 4*(i % 4) .. +3 of a 4 x 16 patch; the load returns to lane L the four rows of
// column L.  Block b of the wave covers columns 16*(b % 2) .. +15 and
// contraction rows 8*(b / 2) .. +7 (in two patches of four rows).
typedef __attribute__((address_space(3))) s16x4_t *lds_patch_t;
__device__ __forceinline__ int transposed_offset(int stride, int col0, int kk0, int lane) {  // elements
    const int blk = lane >> 4, i = lane & 15;
    return (kk0 + ((blk >> 1) << 3) + (i >> 2)) * stride + col0 + ((blk & 1) << 4) + ((i & 3) << 2);
}
__device__ __forceinline__ bf16x8_t frag_transposed(lds_patch_t rows, lds_patch_t next_four) {
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(rows);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(next_four);
    union {
        s16x8_t s;
        bf16x8_t v;
    } out;
    out.s = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return out.v;
}
__device__ __forceinline__ bf16x8_t frag_transposed(const bf16_t *tile, int stride, int col0, int kk0, int lane) {
    const int blk = lane >> 4, i = lane & 15;
    const bf16_t *p = tile + (kk0 + ((blk >> 1) << 3) + (i >> 2)) * stride + col0 + ((blk & 1) << 4) + ((i & 3) << 2);
    return frag_transposed((lds_patch_t)(p), (lds_patch_t)(p + 4 * stride));
}

}  // namespace

}  // namespace rmm
