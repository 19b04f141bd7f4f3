// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nn_compact.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nn_compact) {
    return pass.sketch.cfg == SK_NARROW64 ? launch_pair_tiles<ShapeCompact, B_NCONTIG, ShapeSkNarrow64>(pass, kind, ga, gb, stream, gc)
                                 : hipErrorInvalidValue;
}

}  // namespace rmm
