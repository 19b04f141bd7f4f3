// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nn_compact.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nn_compact) {
    return sk_cfg == SK_NARROW64 ? launch_pair_tiles<ShapeCompact, B_NCONTIG, ShapeSkNarrow64>(kind, ga, gb, blocks_a, tiles_b, shares, stream, gc)
                                 : hipErrorInvalidValue;
}

}  // namespace rmm
