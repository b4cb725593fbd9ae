// Products of several K segments with A k-contiguous, B k-strided (forward) (gemm_layouts.h).
#include "gemm_layouts.h"

namespace dapple {

hipError_t launch_mfma_nt_pack(const GemmArgs& g, const GemmLaunch& l) { return launch_rows<true, true>(g, l, nullptr); }

}  // namespace dapple
