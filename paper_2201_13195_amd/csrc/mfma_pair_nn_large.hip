// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nn_large.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nn_large) {
    return launch_pair_impl<ShapeLarge, B_NCONTIG>(sk_cfg, kind, ga, gb, blocks_a, tiles_b, shares, stream, gc);
}

hipError_t launch_pair_nn(const PairPlain &plain, int sk_cfg, int kind, const GemmArgs &ga, const GemmArgs &gb, int tiles_b,
                          int shares, hipStream_t stream, const ColsumArgs *gc) {
    switch (dx_cfg(plain.cfg, ga.K)) {
        case GEMM_LARGE: return launch_pair_nn_large(sk_cfg, kind, ga, gb, plain.tiles, tiles_b, shares, stream, gc);
        case GEMM_SPLIT: return launch_pair_nn_split(sk_cfg, kind, ga, gb, plain.tiles, tiles_b, shares, stream, gc);
        case GEMM_COMPACT: return launch_pair_nn_compact(sk_cfg, kind, ga, gb, plain.tiles, tiles_b, shares, stream, gc);
        default: return launch_pair_nn_mid(sk_cfg, kind, ga, gb, plain.tiles, tiles_b, shares, stream, gc);
    }
}

}  // namespace rmm
