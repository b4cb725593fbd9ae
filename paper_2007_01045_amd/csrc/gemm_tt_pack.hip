// Products of several K segments with both operands k-strided (weight gradients) (gemm_layouts.h).
#include "gemm_layouts.h"

namespace dapple {

hipError_t launch_mfma_tt_pack(const GemmArgs& g, const GemmLaunch& l) { return launch_tt<true>(g, l, nullptr); }

}  // namespace dapple
