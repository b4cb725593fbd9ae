// Products with both operands k-strided (weight gradients) (gemm_mfma.h).
#include "gemm_mfma.h"

namespace dapple {

hipError_t launch_mfma_tt(int tile, bool short_k, const GemmArgs& g, hipStream_t st) {
  (void)short_k;   // k rows beyond the end read as zero: any K
  const bool bsum = (g.epi & EPI_BSUM) != 0;
  if (g.epi & EPI_SEGACC) {
    switch (tile) {
      case 5:
        return bsum ? launch_mfma<128, 128, 2, 4, 4, true, true, 32, true, false, true>(g, st)
                    : launch_mfma<128, 128, 2, 4, 4, true, true, 32, false, false, true>(g, st);
      case 4:
        return bsum ? launch_mfma<128, 64, 2, 2, 3, true, true, 64, true, false, true>(g, st)
                    : launch_mfma<128, 64, 2, 2, 3, true, true, 64, false, false, true>(g, st);
      default:
        return bsum ? launch_mfma<64, 64, 2, 2, 4, true, true, 64, true, false, true>(g, st)
                    : launch_mfma<64, 64, 2, 2, 4, true, true, 64, false, false, true>(g, st);
    }
  }
  switch (tile) {
    case 1: return launch_mfma<256, 256, 2, 4, 4, true, true, 32>(g, st);
    case 2: return launch_mfma<256, 128, 4, 2, 3, true, true, 64>(g, st);
    case 3:
      return bsum ? launch_mfma<128, 128, 2, 4, 2, true, true, 64, true>(g, st)
                  : launch_mfma<128, 128, 2, 4, 2, true, true, 64>(g, st);
    case 4:
      return bsum ? launch_mfma<128, 64, 2, 2, 3, true, true, 64, true>(g, st)
                  : launch_mfma<128, 64, 2, 2, 3, true, true, 64>(g, st);
    case 5:
      return bsum ? launch_mfma<128, 128, 2, 4, 4, true, true, 32, true>(g, st)
                  : launch_mfma<128, 128, 2, 4, 4, true, true, 32>(g, st);
    case 6: return launch_mfma<128, 128, 2, 4, 5, true, true, 64>(g, st);
    default:
      return bsum ? launch_mfma<64, 64, 2, 2, 4, true, true, 64, true>(g, st)
                  : launch_mfma<64, 64, 2, 2, 4, true, true, 64>(g, st);
  }
}

}  // namespace dapple
