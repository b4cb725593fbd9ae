// The weight gradients of a layer in one launch (gemm_mfma.h's kernel over a list of products).
//
// A layer's three launches (dW2; dW1; dWq, dWk, dWv, dWo) have 256 tiles of 128x128 each at hidden 1024: one per unit,
// so every unit pays a launch's first-tile latency and epilogue three times with nothing beside them, and a tile alone
// on its unit needs eight waves, whose 64x32 parts LDS can feed to half of the matrix peak only.  As one launch of 768
// tiles two workgroups of four waves (64x64 each: 2/3 of the peak) share a unit and hide each other's ends:
// K = 4096 (two micro-batches of 2048 rows) 135 -> 102 us, K = 2048 77 -> 57 us.
#include "gemm_mfma.h"
#include "reduce_jobs.h"

namespace dapple {

struct TileTable {
  int first[WgradGroup::MAX + 1];   // first workgroup of each problem
};

template <int BM, int BN, int WGM, int WGN, int NS, int BK, bool SEG>
__global__ __launch_bounds__(64 * WGM * WGN, SEG ? 2 : 1) void wgrad_group_kernel(WgradGroup w, TileTable t) {
  if ((int)blockIdx.x >= t.first[w.n]) {   // behind the products' tiles: the sums
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int b = blockIdx.x - t.first[w.n], per = (w.jobs.j[0].cols + 63) / 64;
    reduce_columns(w.jobs.j[b / per], w.jobs.nmb, w.jobs.mb_stride, b % per, WGM * WGN / 4, (float(*)[64])smem);
    return;
  }
  int i = 0;
#pragma unroll
  for (int k = 1; k < WgradGroup::MAX; ++k) i += k < w.n && (int)blockIdx.x >= t.first[k];
  // the problem's fields picked with constant indices (a variable index would move the list to scratch memory)
  GemmArgs g{};
  int first = 0;
#pragma unroll
  for (int k = 0; k < WgradGroup::MAX; ++k)
    if (i == k) {
      const WgradProblem& p = w.p[k];
      g.A = p.A; g.B = p.B; g.C = p.C; g.bsum = p.bsum;
      g.M = p.M; g.N = p.N; g.lda = p.lda; g.ldb = p.ldb; g.ldc = p.ldc;
      first = t.first[k];
    }
  g.m_valid = g.M; g.n_valid = g.N; g.K = g.k_valid = w.K; g.kseg_len = w.kseg;
  g.segA = (long)w.kseg * g.lda; g.segB = (long)w.kseg * g.ldb;
  g.epi = EPI_ACC32 | (g.bsum ? EPI_BSUM : 0);
  gemm_mfma_tile<BM, BN, WGM, WGN, NS, true, true, BK, true, false, SEG>(g, (g.M + BM - 1) / BM, (g.N + BN - 1) / BN,
                                                                          blockIdx.x - first, 0);
}

template <int BM, int BN, int WGM, int WGN, int NS, int BK, bool SEG>
static hipError_t launch(const WgradGroup& w, hipStream_t st) {
  typedef GemmTile<BM, BN, WGM, WGN, NS, true, true, BK, false, SEG> CFG;
  auto kern = wgrad_group_kernel<BM, BN, WGM, WGN, NS, BK, SEG>;
  static const hipError_t attr_rc = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                        (int)CFG::LDS_BYTES);
  if (attr_rc != hipSuccess) return attr_rc;
  TileTable t{};
  for (int i = 0; i < w.n; ++i)
    t.first[i + 1] = t.first[i] + ((w.p[i].M + BM - 1) / BM) * ((w.p[i].N + BN - 1) / BN);
  hipLaunchKernelGGL(kern, dim3(t.first[w.n] + w.job_blocks()), dim3(CFG::NT), CFG::LDS_BYTES, st, w, t);
  return hipGetLastError();
}

hipError_t launch_wgrad_group_mfma(const WgradGroup& w, hipStream_t st) {
  long t128 = 0, t12864 = 0;
  for (int i = 0; i < w.n; ++i) {
    t128 += (long)((w.p[i].M + 127) / 128) * ((w.p[i].N + 127) / 128);
    t12864 += (long)((w.p[i].M + 127) / 128) * ((w.p[i].N + 63) / 64);
  }
  const bool seg = w.K > w.kseg;
  const int U = w.units > 0 ? w.units : 256;
  // enough 128x128 tiles for one and a half per unit: four waves, two workgroups per unit; for three quarters of the
  // units: eight waves; else smaller tiles
  if (2 * t128 >= 3 * U) return seg ? launch<128, 128, 2, 2, 4, 32, true>(w, st) : launch<128, 128, 2, 2, 4, 32, false>(w, st);
  if (4 * t128 >= 3 * U) return seg ? launch<128, 128, 2, 4, 4, 32, true>(w, st) : launch<128, 128, 2, 4, 4, 32, false>(w, st);
  if (4 * t12864 >= 3 * U) return seg ? launch<128, 64, 2, 2, 3, 64, true>(w, st) : launch<128, 64, 2, 2, 3, 64, false>(w, st);
  return seg ? launch<64, 64, 2, 2, 4, 64, true>(w, st) : launch<64, 64, 2, 2, 4, 64, false>(w, st);
}

}  // namespace dapple
