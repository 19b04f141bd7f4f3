// Host-side interface between mfma.hip (kernel selection, single launches) and the translation
// units that hold the paired-launch kernels (mfma_pair_*.hip; separate files only to keep the
// build parallel).
#pragma once
#include "mfma_kernels.hpp"

namespace rmm {

// One launch for a plain product (`ga`; nt: Y = X W^T, nn: dX = dY W) and a sketch product (`gb`).
// `gc`, if not null, adds the column blocks of a column-sum problem (colsum.hpp) behind the sketch work-groups.
// `pass` says which tiles, and which of the two comes first in the grid.
hipError_t launch_pair_nt(const PassPlan &pass, int kind, const GemmArgs &ga, const GemmArgs &gb, hipStream_t stream,
                          const ColsumArgs *gc = nullptr);
hipError_t launch_pair_nn(const PassPlan &pass, int kind, const GemmArgs &ga, const GemmArgs &gb, hipStream_t stream,
                          const ColsumArgs *gc = nullptr);
// (one translation unit for each plain tile)
#define RMM_PAIR_DECL(NAME)                                                                                               \
    hipError_t launch_pair_##NAME(const PassPlan &pass, int kind, const GemmArgs &ga, const GemmArgs &gb, hipStream_t stream, \
                                  const ColsumArgs *gc)
RMM_PAIR_DECL(nt_large);
RMM_PAIR_DECL(nt_wide);
RMM_PAIR_DECL(nt_mid);
RMM_PAIR_DECL(nt_compact);
RMM_PAIR_DECL(nn_large);
RMM_PAIR_DECL(nn_wide);
RMM_PAIR_DECL(nn_split);
RMM_PAIR_DECL(nn_mid);
RMM_PAIR_DECL(nn_compact);

// The same for the SORS sketch kind (mfma_pair_sors.hip): `gs` describes the sketch product, whose
// strips stand in the grid as plan.order says (not SORS_APART); row_indexed_b says whether the plain product is dX = dY W (true) or
// Y = X W^T (false).
struct SorsArgs;
hipError_t launch_pair_sors(const SorsPlan &plan, bool row_indexed_b, const GemmArgs &ga, const SorsArgs &gs, hipStream_t stream);

// Shared bodies of launch_pair_{nt,nn}_*.
template <typename SA, int BMODE_A, typename SB>
hipError_t launch_pair_tiles(const PassPlan &pass, int kind, const GemmArgs &ga, const GemmArgs &gb, hipStream_t stream, const ColsumArgs *gc) {
    const int blocks_a = pass.plain.tiles, tiles_b = (int)pass.sketch.tiles, shares = pass.sketch.shares(), sketch_first = pass.sketch_first ? 1 : 0;
    const ColsumArgs c = gc != nullptr ? *gc : ColsumArgs{};
    const int col_blocks = gc != nullptr ? (int)colsum_blocks(c.d, 2) : 0;
    const unsigned grid = (unsigned)(blocks_a + shares + col_blocks);
    if (kind == 0)
        gemm_pair_kernel<SA, BMODE_A, SB, 0><<<grid, SA::THREADS, 0, stream>>>(ga, gb, blocks_a, tiles_b, shares, col_blocks, sketch_first, c);
    else
        gemm_pair_kernel<SA, BMODE_A, SB, 1><<<grid, SA::THREADS, 0, stream>>>(ga, gb, blocks_a, tiles_b, shares, col_blocks, sketch_first, c);
    return hipGetLastError();
}

template <typename SA, int BMODE_A>
hipError_t launch_pair_impl(const PassPlan &pass, int kind, const GemmArgs &ga, const GemmArgs &gb, hipStream_t stream, const ColsumArgs *gc) {
    switch (pass.sketch.cfg) {
        case SK_WIDE: return launch_pair_tiles<SA, BMODE_A, ShapeSkWide>(pass, kind, ga, gb, stream, gc);
        case SK_WIDE64: return launch_pair_tiles<SA, BMODE_A, ShapeSkWide64>(pass, kind, ga, gb, stream, gc);
        case SK_MID64: return launch_pair_tiles<SA, BMODE_A, ShapeSkMid64>(pass, kind, ga, gb, stream, gc);
        case SK_MID: return launch_pair_tiles<SA, BMODE_A, ShapeSkMid>(pass, kind, ga, gb, stream, gc);
        case SK_NARROW64: return launch_pair_tiles<SA, BMODE_A, ShapeSkNarrow64>(pass, kind, ga, gb, stream, gc);
        case SK_NARROW: return launch_pair_tiles<SA, BMODE_A, ShapeSkNarrow>(pass, kind, ga, gb, stream, gc);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rmm
