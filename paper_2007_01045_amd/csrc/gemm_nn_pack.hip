// Products of several K segments with both operands k-contiguous (data gradients) (gemm_layouts.h).
#include "gemm_layouts.h"

namespace dapple {

hipError_t launch_mfma_nn_pack(const GemmArgs& g, const GemmLaunch& l) { return launch_rows<false, true>(g, l, nullptr); }

}  // namespace dapple
