// The launches of gemm_mfma_kernel per operand layout (gemm_mfma.h), each layout twice: PACK or not, in files of their own.
#pragma once
#include "gemm_mfma.h"

namespace dapple {

// (A tile that a layout does not hold is an error: choose_tile names none.)

// A k-contiguous: forward products (BKS) and data gradients
template <bool BKS, bool PACK>
static hipError_t launch_rows(const GemmArgs& g, const GemmLaunch& l, LaunchMfma packed) {
  if (l.short_k)   // K segments that are no multiple of 64: the masked variants
    return l.tile == 3 ? launch_mfma<128, 128, 2, 4, 2, false, BKS, 64, PACK, false, true>(g, l, packed)
                       : launch_mfma<128, 64, 4, 2, 3, false, BKS, 64, PACK, false, true>(g, l, packed);
  switch (l.tile) {
    case 1: return launch_mfma<256, 256, 2, 4, 4, false, BKS, 32, PACK>(g, l, packed);
    case 2: return launch_mfma<256, 128, 4, 2, 3, false, BKS, 64, PACK>(g, l, packed);
    case 3: return launch_mfma<128, 128, 2, 4, 2, false, BKS, 64, PACK>(g, l, packed);
    case 4: return launch_mfma<128, 64, 4, 2, 3, false, BKS, 64, PACK>(g, l, packed);
    case 6: return launch_mfma<128, 128, 2, 4, 5, false, BKS, 64, PACK>(g, l, packed);
    case 8: return launch_mfma<128, 128, 2, 2, 4, false, BKS, 32, PACK>(g, l, packed);
    case 9: return launch_mfma<32, 64, 1, 2, 4, false, BKS, 64, PACK>(g, l, packed);
    case 10: return launch_mfma<32, 32, 1, 1, 4, false, BKS, 64, PACK>(g, l, packed);
    case 12: return launch_mfma<128, 64, 4, 2, 4, false, BKS, 64, PACK>(g, l, packed);
    case 7: return launch_mfma<64, 64, 2, 2, 4, false, BKS, 64, PACK>(g, l, packed);
    default: return hipErrorInvalidValue;
  }
}

// A k-strided, B k-contiguous: no product of the stage, dapple_gemm alone has them
template <bool PACK>
static hipError_t launch_tn(const GemmArgs& g, const GemmLaunch& l, LaunchMfma packed) {
  if (l.short_k)
    return l.tile == 3 ? launch_mfma<128, 128, 2, 4, 2, true, false, 64, PACK, false, true>(g, l, packed)
                       : launch_mfma<128, 64, 2, 2, 3, true, false, 64, PACK, false, true>(g, l, packed);
  switch (l.tile) {
    case 1: return launch_mfma<256, 256, 2, 4, 4, true, false, 32, PACK>(g, l, packed);
    case 2: return launch_mfma<256, 128, 4, 2, 3, true, false, 64, PACK>(g, l, packed);
    case 3: return launch_mfma<128, 128, 2, 4, 2, true, false, 64, PACK>(g, l, packed);
    case 4: return launch_mfma<128, 64, 2, 2, 3, true, false, 64, PACK>(g, l, packed);
    case 6: return launch_mfma<128, 128, 2, 4, 5, true, false, 64, PACK>(g, l, packed);
    case 7: return launch_mfma<64, 64, 2, 2, 4, true, false, 64, PACK>(g, l, packed);
    default: return hipErrorInvalidValue;
  }
}

// Both k-strided: weight gradients.  (k rows beyond the end read as zero: any K.)
template <bool PACK>
static hipError_t launch_tt(const GemmArgs& g, const GemmLaunch& l, LaunchMfma packed) {
  const bool bsum = (g.epi & EPI_BSUM) != 0;
  if constexpr (!PACK)
    if (g.epi & EPI_SEGACC) {
      switch (l.tile) {
        case 5:
          return bsum ? launch_mfma<128, 128, 2, 4, 4, true, true, 32, false, true, false, true>(g, l, packed)
                      : launch_mfma<128, 128, 2, 4, 4, true, true, 32, false, false, false, true>(g, l, packed);
        case 4:
          return bsum ? launch_mfma<128, 64, 2, 2, 3, true, true, 64, false, true, false, true>(g, l, packed)
                      : launch_mfma<128, 64, 2, 2, 3, true, true, 64, false, false, false, true>(g, l, packed);
        case 7:
          return bsum ? launch_mfma<64, 64, 2, 2, 4, true, true, 64, false, true, false, true>(g, l, packed)
                      : launch_mfma<64, 64, 2, 2, 4, true, true, 64, false, false, false, true>(g, l, packed);
        default: return hipErrorInvalidValue;
      }
    }
  switch (l.tile) {
    case 1: return launch_mfma<256, 256, 2, 4, 4, true, true, 32, PACK>(g, l, packed);
    case 2: return launch_mfma<256, 128, 4, 2, 3, true, true, 64, PACK>(g, l, packed);
    case 3:
      return bsum ? launch_mfma<128, 128, 2, 4, 2, true, true, 64, PACK, true>(g, l, packed)
                  : launch_mfma<128, 128, 2, 4, 2, true, true, 64, PACK>(g, l, packed);
    case 4:
      return bsum ? launch_mfma<128, 64, 2, 2, 3, true, true, 64, PACK, true>(g, l, packed)
                  : launch_mfma<128, 64, 2, 2, 3, true, true, 64, PACK>(g, l, packed);
    case 5:
      return bsum ? launch_mfma<128, 128, 2, 4, 4, true, true, 32, PACK, true>(g, l, packed)
                  : launch_mfma<128, 128, 2, 4, 4, true, true, 32, PACK>(g, l, packed);
    case 6: return launch_mfma<128, 128, 2, 4, 5, true, true, 64, PACK>(g, l, packed);
    case 7:
      return bsum ? launch_mfma<64, 64, 2, 2, 4, true, true, 64, PACK, true>(g, l, packed)
                  : launch_mfma<64, 64, 2, 2, 4, true, true, 64, PACK>(g, l, packed);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dapple
