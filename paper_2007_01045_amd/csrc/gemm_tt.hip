// Products with both operands k-strided (weight gradients) (gemm_layouts.h).
#include "gemm_layouts.h"

namespace dapple {

hipError_t launch_mfma_tt(const GemmArgs& g, const GemmLaunch& l) { return launch_tt<false>(g, l, launch_mfma_tt_pack); }

}  // namespace dapple
