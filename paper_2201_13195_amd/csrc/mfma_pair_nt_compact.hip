// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nt_compact.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nt_compact) {
    return pass.sketch.cfg == SK_NARROW64 ? launch_pair_tiles<ShapeCompact, B_KCONTIG, ShapeSkNarrow64>(pass, kind, ga, gb, stream, gc)
                                 : hipErrorInvalidValue;
}

}  // namespace rmm
