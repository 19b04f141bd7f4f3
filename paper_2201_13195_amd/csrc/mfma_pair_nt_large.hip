// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nt_large.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nt_large) {
    return launch_pair_impl<ShapeLarge, B_KCONTIG>(sk_cfg, kind, ga, gb, blocks_a, tiles_b, shares, stream, gc);
}

hipError_t launch_pair_nt(const PairPlain &plain, int sk_cfg, int kind, const GemmArgs &ga, const GemmArgs &gb, int tiles_b,
                          int shares, hipStream_t stream, const ColsumArgs *gc) {
    switch (plain.cfg) {
        case GEMM_LARGE: return launch_pair_nt_large(sk_cfg, kind, ga, gb, plain.tiles, tiles_b, shares, stream, gc);
        case GEMM_COMPACT: return launch_pair_nt_compact(sk_cfg, kind, ga, gb, plain.tiles, tiles_b, shares, stream, gc);
        default: return launch_pair_nt_mid(sk_cfg, kind, ga, gb, plain.tiles, tiles_b, shares, stream, gc);
    }
}

}  // namespace rmm
