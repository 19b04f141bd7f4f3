// Instantiations of plain_pass_kernel (see plain_pass.hpp).
#include "plain_pass.hpp"

namespace rmm {

hipError_t launch_backward_pass_bf16x8_(const PlainLaunch &p, hipStream_t stream) {
    return launch_plain_pass_rows<bf16_t, 4, 3, PB_N>(p, stream);
}

}  // namespace rmm
