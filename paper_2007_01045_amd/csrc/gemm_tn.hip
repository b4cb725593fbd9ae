// Products with A k-strided and B k-contiguous (gemm_layouts.h).
#include "gemm_layouts.h"

namespace dapple {

hipError_t launch_mfma_tn(const GemmArgs& g, const GemmLaunch& l) { return launch_tn<false>(g, l, launch_mfma_tn_pack); }

}  // namespace dapple
