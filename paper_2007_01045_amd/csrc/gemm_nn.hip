// Products with both operands k-contiguous (data gradients) (gemm_mfma.h).
#include "gemm_mfma.h"

namespace dapple {

hipError_t launch_mfma_nn(int tile, bool short_k, const GemmArgs& g, hipStream_t st) {
  if (short_k)   // K segments that are no multiple of 64: the masked variants
    return tile == 3 ? launch_mfma<128, 128, 2, 4, 2, false, false, 64, false, true>(g, st)
                     : launch_mfma<128, 64, 2, 2, 3, false, false, 64, false, true>(g, st);
  switch (tile) {
    case 1: return launch_mfma<256, 256, 2, 4, 4, false, false, 32>(g, st);
    case 2: return launch_mfma<256, 128, 4, 2, 3, false, false, 64>(g, st);
    case 3: return launch_mfma<128, 128, 2, 4, 2, false, false, 64>(g, st);
    case 4: return launch_mfma<128, 64, 2, 2, 3, false, false, 64>(g, st);
    case 6: return launch_mfma<128, 128, 2, 4, 5, false, false, 64>(g, st);
    case 8: return launch_mfma<128, 128, 2, 2, 4, false, false, 32>(g, st);
    case 9: return launch_mfma<32, 64, 1, 2, 4, false, false, 64>(g, st);
    case 10: return launch_mfma<32, 32, 1, 1, 4, false, false, 64>(g, st);
    default: return launch_mfma<64, 64, 2, 2, 4, false, false, 64>(g, st);
  }
}

}  // namespace dapple
