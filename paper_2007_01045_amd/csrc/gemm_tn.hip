// Products with A k-strided and B k-contiguous (gemm_mfma.h): no product of the stage, dapple_gemm alone has them.
#include "gemm_mfma.h"

namespace dapple {

hipError_t launch_mfma_tn(int tile, bool short_k, const GemmArgs& g, hipStream_t st) {
  if (short_k)   // K segments that are no multiple of 64: the masked variants
    return tile == 3 ? launch_mfma<128, 128, 2, 4, 2, true, false, 64, false, true>(g, st)
                     : launch_mfma<128, 64, 2, 2, 3, true, false, 64, false, true>(g, st);
  switch (tile) {
    case 1: return launch_mfma<256, 256, 2, 4, 4, true, false, 32>(g, st);
    case 2: return launch_mfma<256, 128, 4, 2, 3, true, false, 64>(g, st);
    case 3: return launch_mfma<128, 128, 2, 4, 2, true, false, 64>(g, st);
    case 4: return launch_mfma<128, 64, 2, 2, 3, true, false, 64>(g, st);
    case 6: return launch_mfma<128, 128, 2, 4, 5, true, false, 64>(g, st);
    default: return launch_mfma<64, 64, 2, 2, 4, true, false, 64>(g, st);
  }
}

}  // namespace dapple
