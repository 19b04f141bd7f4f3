// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nt_wide.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nt_wide) {
    return launch_pair_impl<ShapeWide, B_KCONTIG>(pass, kind, ga, gb, stream, gc);
}

}  // namespace rmm
