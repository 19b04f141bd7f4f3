// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nn_split.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nn_split) {
    return launch_pair_impl<ShapeSplit, B_NCONTIG>(pass, kind, ga, gb, stream, gc);
}

}  // namespace rmm
