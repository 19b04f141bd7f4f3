// Instantiations of plain_pass_kernel (see plain_pass.hpp), and the forward pass whose Y runs on the tiles of mfma_kernels.hpp.
#include "mfma_kernels.hpp"
#include "plain_pass.hpp"

namespace rmm {

namespace {

// X and W have rows on 16 bytes and only Y has not: the tiles of Y load as those of even widths do, straight into LDS, and write rows that start
// anywhere (OUT_BF16_ANY).  Beside the sketch tiles of plain_kernels.hpp, whose entries keep their fp32 precision; either takes half
// of a compute unit.  What bounds the launch at 3000 x 768 -> 1001, k = 300, is now those sketch tiles, which generate (22 us; Y alone 13.6).
template <typename S, typename SS, int SKETCH>
__global__ void __launch_bounds__(kPlainThreads, 4) forward_any_width_kernel(GemmArgs ga, PlainArgs gs, int plain_blocks, int sketch_blocks) {
    constexpr int BS = PlainTile<bf16_t, SS, SKETCH, PB_N>::LDS_BYTES, BYTES = S::LDS_BYTES > BS ? S::LDS_BYTES : BS;
    static_assert(S::THREADS == kPlainThreads && BYTES <= 80 * 1024, "two work-groups on a compute unit");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[BYTES];
    const int b = (int)blockIdx.x;
    if (b < sketch_blocks)
        plain_tile<bf16_t, bf16_t, SS, SKETCH, PB_N, 4, 4>(gs, reinterpret_cast<bf16_t *>(lds), b, sketch_blocks);
    else
        gemm_tile<S, A_KCONTIG, B_KCONTIG, OUT_BF16_ANY>(ga, reinterpret_cast<bf16_t *>(lds), b - sketch_blocks, plain_blocks);
}

template <typename S, typename SS>
hipError_t launch_any_width(const PlainLaunch &p, const GemmArgs &g, hipStream_t stream) {
    const int tiles = (int)tiles_of(g.M, g.N, S::BM, S::BN);
    const unsigned grid = (unsigned)(tiles + p.sketch_blocks);
    if (p.gs.kind == 0)
        forward_any_width_kernel<S, SS, PA_GAUSS><<<grid, kPlainThreads, 0, stream>>>(g, p.gs, tiles, p.sketch_blocks);
    else
        forward_any_width_kernel<S, SS, PA_SIGN><<<grid, kPlainThreads, 0, stream>>>(g, p.gs, tiles, p.sketch_blocks);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_forward_pass_bf16x8(const PlainLaunch &p, hipStream_t stream) {
    const int tile = p.plain_blocks > 0 ? p.tile : -1;
    if (tile < 0) return launch_plain_pass_rows<bf16_t, 4, 4, PB_K>(p, stream);
    GemmArgs g{};
    g.A = (const bf16_t *)p.ga.A, g.lda = p.ga.lda, g.B = (const bf16_t *)p.ga.B, g.ldb = p.ga.ldb, g.C = p.ga.C, g.ldc = p.ga.ldc;
    g.bias = (const bf16_t *)p.ga.bias, g.M = p.ga.M, g.N = p.ga.N, g.K = p.ga.K, g.alpha = p.ga.alpha;
    if (tile == GEMM_COMPACT)  // (in place of 128 x 128 tiles, beside which no sketch tiles are 32 x 32)
        return p.sketch_small ? hipErrorInvalidValue : launch_any_width<ShapeCompact, PlainSketch>(p, g, stream);
    return p.sketch_small ? launch_any_width<ShapeFlat, PlainTiny>(p, g, stream) : launch_any_width<ShapeFlat, PlainSketch>(p, g, stream);
}

}  // namespace rmm
