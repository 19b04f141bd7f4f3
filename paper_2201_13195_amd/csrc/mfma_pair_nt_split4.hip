// Paired-launch kernels (see mfma_pair.hpp): launch_pair_nt_split4.
#include "mfma_pair.hpp"

namespace rmm {

RMM_PAIR_DECL(nt_split4) {
    return launch_pair_impl<ShapeSplit, B_KCONTIG, 4>(sk_cfg, kind, ga, gb, blocks_a, tiles_b, shares, stream, gc);
}

}  // namespace rmm
