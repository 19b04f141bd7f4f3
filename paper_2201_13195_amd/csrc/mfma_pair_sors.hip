// Paired-launch kernels for the SORS sketch kind: the tiles of a plain product (Y = X W^T or
// dX = dY W) and the strips of the sketch product of the same pass in one grid (plan_sors says which and where).
#include "mfma_pair.hpp"
#include "sors_kernels.hpp"

namespace rmm {

namespace {

constexpr int kPairChunkLog = 11;  // chunks of 2048 tokens, as the strip kernel on its own

template <typename SA, int BMODE_A, bool SUMS>
__global__ void __launch_bounds__(SA::THREADS) gemm_sors_pair_kernel(GemmArgs ga, SorsArgs gs, int blocks_a, int chunks,
                                                                     int sors_first) {
    typedef StripShape<kPairChunkLog> SS;
    static_assert(SA::THREADS == 512, "two strips of 256 threads");
    constexpr int BYTES_A = SA::LDS_BYTES, PLANE_BYTES = 2 * SS::REGION * 16;
    constexpr int BYTES_S = PLANE_BYTES + 1024 * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[BYTES_A > BYTES_S ? BYTES_A : BYTES_S];
    // The strips come last in the grid when they are to fill the compute units the plain product's
    // last round leaves idle, first when the plain product runs several full rounds and the (long)
    // strips should start with it rather than after it.
    const int strips = (int)gridDim.x - blocks_a;
    const int plain = sors_first ? (int)blockIdx.x - strips : (int)blockIdx.x;
    if (plain >= 0 && plain < blocks_a)
        gemm_tile<SA, A_KCONTIG, BMODE_A, OUT_BF16>(ga, reinterpret_cast<bf16_t *>(lds), plain, blocks_a);
    else
        sors_strip_body<kPairChunkLog, true, 2, 8, SUMS>(gs, chunks, reinterpret_cast<float4 *>(lds),
                                                reinterpret_cast<uint32_t *>(lds + PLANE_BYTES),
                                                sors_first ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - blocks_a, strips, 1, gs.k);
}

// Tiles of 128 x 128 in half of a compute unit's LDS and registers, strips in the other half or in what the tiles leave.  What bounds a tile
// is the way of its operands into LDS, what bounds a strip vector additions and LDS passes between barriers: beside each other either
// waits less.  The tiles come first: they are the longer ones, and the strips fill the places behind them.
// The strips as the strip kernel has them alone: LC = 10 and 11 all tokens at once, ACC chunks of 2048 with accumulators.  Up to 512
// tokens too take 1024 points, whose work-groups have as many waves as those of the tiles; the upper half is zeros, and the results the same.
template <int BMODE_A, int LC, bool ACC, bool SUMS>
__global__ void __launch_bounds__(512, 4) gemm_sors_compact_kernel(GemmArgs ga, SorsArgs gs, int tiles, int chunks) {
    constexpr int BYTES_A = ShapeCompact::LDS_BYTES, PLANE_BYTES = StripShape<LC>::REGION * 16, BYTES_S = PLANE_BYTES + 1024 * 4;
    static_assert(ShapeCompact::THREADS == 512 && BYTES_A <= 80 * 1024 && BYTES_S <= 80 * 1024, "two work-groups on a compute unit");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[BYTES_A > BYTES_S ? BYTES_A : BYTES_S];
    const int block = (int)blockIdx.x;
    if (block < tiles)
        gemm_tile<ShapeCompact, A_KCONTIG, BMODE_A, OUT_BF16>(ga, reinterpret_cast<bf16_t *>(lds), block, tiles);
    else
        sors_strip_body<LC, ACC, 1, 8, SUMS>(gs, chunks, reinterpret_cast<float4 *>(lds), reinterpret_cast<uint32_t *>(lds + PLANE_BYTES), block - tiles,
                                             (int)gridDim.x - tiles, 1, gs.k);
}

template <int BMODE_A, int LC, bool ACC>
hipError_t launch_compact(const GemmArgs &ga, const SorsArgs &gs, int tiles, hipStream_t stream) {
    const unsigned grid = (unsigned)(tiles + gs.d / 8);
    const int chunks = sors_chunks(gs.n);
    if constexpr (BMODE_A == B_NCONTIG)
        if (gs.colsum != nullptr) {
            gemm_sors_compact_kernel<BMODE_A, LC, ACC, true><<<grid, 512, 0, stream>>>(ga, gs, tiles, chunks);
            return hipGetLastError();
        }
    gemm_sors_compact_kernel<BMODE_A, LC, ACC, false><<<grid, 512, 0, stream>>>(ga, gs, tiles, chunks);
    return hipGetLastError();
}

template <typename SA, int BMODE_A>
hipError_t launch_impl(const GemmArgs &ga, const SorsArgs &gs, int blocks_a, int chunks, int sors_first, hipStream_t stream) {
    const unsigned strips2 = (unsigned)((gs.d / 8 + 1) / 2);
    const unsigned grid = (unsigned)blocks_a + strips2;
    if constexpr (BMODE_A == B_NCONTIG)
        if (gs.colsum != nullptr) {
            gemm_sors_pair_kernel<SA, BMODE_A, true><<<grid, SA::THREADS, 0, stream>>>(ga, gs, blocks_a, chunks, sors_first);
            return hipGetLastError();
        }
    gemm_sors_pair_kernel<SA, BMODE_A, false><<<grid, SA::THREADS, 0, stream>>>(ga, gs, blocks_a, chunks, sors_first);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_pair_sors(const SorsPlan &plan, bool row_indexed_b, const GemmArgs &ga, const SorsArgs &gs, hipStream_t stream) {
    const PairPlain &plain = plan.plain;
    if (plan.order == SORS_COMPACT) {
        const int l = sors_log(gs.n);
        if (row_indexed_b)
            return l <= 10   ? launch_compact<B_NCONTIG, 10, false>(ga, gs, plain.tiles, stream)
                   : l == 11 ? launch_compact<B_NCONTIG, 11, false>(ga, gs, plain.tiles, stream)
                             : launch_compact<B_NCONTIG, 11, true>(ga, gs, plain.tiles, stream);
        return l <= 10   ? launch_compact<B_KCONTIG, 10, false>(ga, gs, plain.tiles, stream)
               : l == 11 ? launch_compact<B_KCONTIG, 11, false>(ga, gs, plain.tiles, stream)
                         : launch_compact<B_KCONTIG, 11, true>(ga, gs, plain.tiles, stream);
    }
    const int first = plan.order == SORS_FRONT ? 1 : 0, chunks = sors_chunks(gs.n);
#define RMM_SORS_CASE(CFG, SHAPE)                                                                     \
    case CFG:                                                                                         \
        return row_indexed_b ? launch_impl<SHAPE, B_NCONTIG>(ga, gs, plain.tiles, chunks, first, stream) \
                             : launch_impl<SHAPE, B_KCONTIG>(ga, gs, plain.tiles, chunks, first, stream);
    if (row_indexed_b && dx_cfg(plain.cfg, ga.K) == GEMM_SPLIT) return launch_impl<ShapeSplit, B_NCONTIG>(ga, gs, plain.tiles, chunks, first, stream);
    switch (plain.cfg) {
        RMM_SORS_CASE(GEMM_LARGE, ShapeLarge)
        RMM_SORS_CASE(GEMM_MID, ShapeMid)
        default: return hipErrorInvalidValue;
    }
#undef RMM_SORS_CASE
}

}  // namespace rmm
