// Instantiations of plain_pass_kernel (see plain_pass.hpp).
#include "plain_pass.hpp"

namespace rmm {

hipError_t launch_plain_pass_f32x4(const PlainLaunch &p, bool b_rows_k, hipStream_t stream) {
    return launch_plain_pass_impl<float, 4>(p, b_rows_k, stream);
}

}  // namespace rmm
