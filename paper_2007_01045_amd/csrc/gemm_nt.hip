// Products with A k-contiguous, B k-strided (forward) (gemm_layouts.h).
#include "gemm_layouts.h"

namespace dapple {

hipError_t launch_mfma_nt(const GemmArgs& g, const GemmLaunch& l) { return launch_rows<true, false>(g, l, launch_mfma_nt_pack); }

}  // namespace dapple
