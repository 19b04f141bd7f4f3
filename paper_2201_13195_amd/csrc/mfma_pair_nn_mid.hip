// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nn_mid.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nn_mid) {
    return launch_pair_impl<ShapeMid, B_NCONTIG>(pass, kind, ga, gb, stream, gc);
}

}  // namespace rmm
