// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nn_wide.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nn_wide) {
    return launch_pair_impl<ShapeWide, B_NCONTIG>(pass, kind, ga, gb, stream, gc);
}

}  // namespace rmm
