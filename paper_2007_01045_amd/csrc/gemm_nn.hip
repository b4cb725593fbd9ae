// Products with both operands k-contiguous (data gradients) (gemm_layouts.h).
#include "gemm_layouts.h"

namespace dapple {

hipError_t launch_mfma_nn(const GemmArgs& g, const GemmLaunch& l) { return launch_rows<false, false>(g, l, launch_mfma_nn_pack); }

}  // namespace dapple
