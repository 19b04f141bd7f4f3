// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nt_large.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nt_large) {
    return launch_pair_impl<ShapeLarge, B_KCONTIG>(pass, kind, ga, gb, stream, gc);
}

hipError_t launch_pair_nt(const PassPlan &pass, int kind, const GemmArgs &ga, const GemmArgs &gb, hipStream_t stream,
                          const ColsumArgs *gc) {
    switch (pass.plain.cfg) {
        case GEMM_LARGE: return launch_pair_nt_large(pass, kind, ga, gb, stream, gc);
        case GEMM_WIDE: return launch_pair_nt_wide(pass, kind, ga, gb, stream, gc);
        case GEMM_COMPACT: return launch_pair_nt_compact(pass, kind, ga, gb, stream, gc);
        default: return launch_pair_nt_mid(pass, kind, ga, gb, stream, gc);
    }
}

}  // namespace rmm
