// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nt_split.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nt_split) {
    return launch_pair_impl<ShapeSplit, B_KCONTIG>(sk_cfg, kind, ga, gb, blocks_a, tiles_b, shares, stream, gc);
}

}  // namespace rmm
