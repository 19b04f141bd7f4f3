// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nt_mid.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nt_mid) {
    return launch_pair_impl<ShapeMid, B_KCONTIG>(pass, kind, ga, gb, stream, gc);
}

}  // namespace rmm
