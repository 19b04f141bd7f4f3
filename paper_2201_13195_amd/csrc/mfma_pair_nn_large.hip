// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nn_large.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nn_large) {
    return launch_pair_impl<ShapeLarge, B_NCONTIG>(pass, kind, ga, gb, stream, gc);
}

hipError_t launch_pair_nn(const PassPlan &pass, int kind, const GemmArgs &ga, const GemmArgs &gb, hipStream_t stream,
                          const ColsumArgs *gc) {
    switch (dx_cfg(pass.plain.cfg, ga.K)) {
        case GEMM_LARGE: return launch_pair_nn_large(pass, kind, ga, gb, stream, gc);
        case GEMM_WIDE: return launch_pair_nn_wide(pass, kind, ga, gb, stream, gc);
        case GEMM_SPLIT: return launch_pair_nn_split(pass, kind, ga, gb, stream, gc);
        case GEMM_COMPACT: return launch_pair_nn_compact(pass, kind, ga, gb, stream, gc);
        default: return launch_pair_nn_mid(pass, kind, ga, gb, stream, gc);
    }
}

}  // namespace rmm
