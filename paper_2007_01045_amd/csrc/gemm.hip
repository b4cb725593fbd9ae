// GEMM kernels of the stage: every linear layer's forward, data-gradient and
// weight-gradient product is C = epilogue(sum_k A(m,k) B(n,k)) with either operand
// stored k-contiguous or k-strided.
//
//  * gemm_mfma_kernel (gemm_mfma.h): bf16 operands, fp32 accumulation on the gfx950 matrix
//    cores (v_mfma_f32_32x32x16_bf16).  4 or 8 waves in a grid over a
//    BM x BN tile, k-tiles of 64 or 32, an LDS ring of 2 to 5 k-tiles filled by buffer
//    loads that write straight into LDS.  k-contiguous operands sit in LDS as [row][k]
//    and are read with 128-bit loads; k-strided operands sit as [k][rows] and are
//    read with the LDS transpose read, so no transposed copy of an activation or a
//    weight is ever made in HBM (both layouts XOR-swizzled against bank conflicts).  The MFMA is issued with the B fragment as its
//    first operand: each lane then owns 4 consecutive output columns of one
//    output row, which the epilogue stages through LDS into coalesced stores.
//  * gemm_plain_kernel: one thread per output element, fp32 accumulation in k
//    order; used for shapes neither the MFMA kernel nor the fp32 kernels (gemm_f32.hip) take.
#include <type_traits>
#include <utility>

#include "device_common.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace dapple {

// ------------------------------------------------------------------ plain kernel
__device__ __forceinline__ void plain_bsum(const GemmArgs& g, int z, int col, float t) {
  if (z == 0 && g.bsum) g.bsum[col] += t;
}

template <typename T>
__global__ void gemm_plain_kernel(GemmArgs g) {
  int col = blockIdx.x * blockDim.x + threadIdx.x;
  int row = blockIdx.y * blockDim.y + threadIdx.y;
  int z = blockIdx.z;
  if (row >= g.M || col >= g.N) return;
  const T *A = (const T*)g.A + z * g.sA, *B = (const T*)g.B + z * g.sB;
  float acc = 0.f, bsum = 0.f;
  int nseg = g.K / g.kseg_len;
  const bool segacc = (g.epi & EPI_SEGACC) != 0;
  for (int s = 0; s < nseg; ++s) {
    if (segacc && s) {   // the segment before is complete
      epilogue_store<T>(g, z * g.sC, z * g.sBias, row, col, acc);
      if ((g.epi & EPI_BSUM) && row == 0) plain_bsum(g, z, col, bsum);
      acc = bsum = 0.f;
    }
    const T* As = A + s * g.segA;
    const T* Bs = B + s * g.segB;
    for (int k = 0; k < g.kseg_len; ++k) {
      if (k >= g.k_valid) break;
      float a = row < g.m_valid ? to_f32(g.a_kstrided ? As[(long)k * g.lda + row] : As[(long)row * g.lda + k]) : 0.f;
      float b = col < g.n_valid ? to_f32(g.b_kstrided ? Bs[(long)k * g.ldb + col] : Bs[(long)col * g.ldb + k]) : 0.f;
      acc = fmaf(a, b, acc);
      bsum += b;
    }
  }
  if ((g.epi & EPI_BSUM) && row == 0) plain_bsum(g, z, col, bsum);
  epilogue_store<T>(g, z * g.sC, z * g.sBias, row, col, acc);
}

// ------------------------------------------------------------------ host side
static bool aligned_to(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

bool gemm_uses_mfma(Dtype dt, const GemmArgs& g) {
  if (dt != DT_BF16) return false;
  constexpr int BK = 64;  // the widest k-tile
  if (g.K < 1 || g.kseg_len < 1 || g.K % g.kseg_len) return false;
  // a k-contiguous operand is read in chunks of 8 elements, so a segment's end must fall between two chunks; with
  // both operands k-strided K may be anything
  if (g.kseg_len % 8 && !(g.a_kstrided && g.b_kstrided)) return false;
  if (g.lda % 8 || g.ldb % 8 || g.ldc % 4 || g.N % 4) return false;
  if (g.sA % 8 || g.sB % 8 || g.sC % 4 || g.sBias % 4 || g.segA % 8 || g.segB % 8) return false;
  if (!aligned_to(g.A, 16) || !aligned_to(g.B, 16) || !aligned_to(g.C, 16)) return false;
  {  // the kernel counts the readable bytes of an operand segment in a 32-bit buffer field
    const int kv = g.k_valid > 0 ? g.k_valid : g.K, mv = g.m_valid > 0 ? g.m_valid : g.M, nv = g.n_valid > 0 ? g.n_valid : g.N;
    const long a_ext = g.a_kstrided ? ((long)(kv - 1) * g.lda + mv) * 2 : ((long)(mv - 1) * g.lda + g.kseg_len) * 2;
    const long b_ext = g.b_kstrided ? ((long)(kv - 1) * g.ldb + nv) * 2 : ((long)(nv - 1) * g.ldb + g.kseg_len) * 2;
    if (a_ext > 0x7fffffffL - 4096 || b_ext > 0x7fffffffL - 4096) return false;
    if ((long)BK * g.lda * 2 > 0x7fffffffL || (long)BK * g.ldb * 2 > 0x7fffffffL) return false;
  }
  if ((g.epi & (EPI_ADD | EPI_MUL | EPI_ROWDOT)) && (g.ldaux % 4 || !aligned_to(g.aux, 16))) return false;
  if ((g.epi & EPI_ROWDOT) && (g.kseg_len % BK || (g.epi & (EPI_ADD | EPI_MUL | EPI_GELU | EPI_ACC32 | EPI_OUT32)) || g.batch != 1 ||
                               !g.rowdot || !g.aux || !aligned_to(g.rowdot, 4)))
    return false;
  if ((g.epi & EPI_AUXLN) && ((g.epi & (EPI_ADD | EPI_AUX32 | EPI_MUL | EPI_ACC32)) != (EPI_ADD | EPI_AUX32) || g.batch != 1 ||
                              !aligned_to(g.ln_gamma, 8) || !aligned_to(g.ln_beta, 8)))
    return false;
  if ((g.epi & EPI_BIAS) && !aligned_to(g.bias, 8)) return false;
  if ((g.epi & EPI_GELU) && !aligned_to(g.C2, 8)) return false;
  if ((g.epi & EPI_BSUM) && !(g.a_kstrided && g.b_kstrided)) return false;
  if ((g.epi & EPI_SEGACC) && !((g.epi & EPI_ACC32) && g.a_kstrided && g.b_kstrided && !(g.epi & (EPI_BIAS | EPI_ADD | EPI_MUL)))) return false;
  return true;
}

// Tile choice.  Every k-tile goes global -> LDS through the compute unit's vector cache at 64 bytes per clock, and from
// LDS to the waves at 128 bytes per clock, against 4096 MFMA flops per clock, so the larger a wave's tile the less LDS
// holds it back (64x32 per wave, the 128x128 tile of 8 waves: half of the matrix peak; 64x64: 73%; 128x64: all of it).
// Against that, a product must reach the 256 units, a k-tile must have been requested long enough ahead (about 1 us
// from HBM: the fewer workgroups share a unit, the deeper the ring has to be), and a launch's fixed cost -- first
// tile's latency, epilogue -- is only hidden by another workgroup on the same unit.  Eight waves (two per SIMD) beat
// four on every tile of 128x128 and up with k-tiles of 64.  Alone, in us (T rows; "->" four waves -> eight where both were measured):
//   1: 256x256, four stages of 32      T=8192 N=4096 K=1024 GELU 112 -> 92, gate 90 (128x128: 101); T=4096 44 and 42
//   2: 256x128, three stages of 64     T=8192 N=1024 K=4096 residual 77 -> 72 (128x128: 84), gradient 81 -> 65
//   3: 128x128, two stages of 64       two workgroups per unit: T=2048 N=4096 K=1024 GELU 26, gate 23 (256x256: 36, 31)
//   4: 128x64, three stages of 64      T=2048 N=1024 K=4096 27 (128x128: 46); T=4096 N=1024 K=1024 17 (20); eight waves of
//                                      32x32 where A is k-contiguous: two per SIMD wait for a k-tile's barrier and its reads
//                                      in each other's time, which is more than the waves of 64x32 save in reads.  T=1800
//                                      N=768 K=3072 forward 20.7 -> 19.4, gradient 20.0 -> 19.0, T=1400 N=1024 K=4096 25.4 ->
//                                      24.5, 24.8 -> 24.1; with more tiles than units T=2560 39.9 -> 39.4, T=3000 N=768 27.5 -> 28.1
//                                      (cold weights 33.3 and 34.7), which iterations do not show: forward products in four waves
//                                      there 0-0.3% slower 512 to 896 wide, 0.2% faster 1024 wide
//   5: 128x128, four stages of 32      weight gradients: both operands k-strided, so a 32-deep tile still reads whole
//                                      256-byte rows, and three tiles are in flight in the LDS of two of 64
//   6: 128x128, five stages of 64      one workgroup per unit: T=4096 N=1024 K=4096 67 -> 45
//   7: 64x64, four stages of 64        T=512 N=1024 K=4096 23 (128x64) -> 16, K=1024 9.6 -> 6.9; T=1024 23 -> 17
//   8: 128x128, four waves, four       two workgroups per unit: T=4096 N=1024 K=1024 17 (128x64: 19)
//      stages of 32
//   9: 32x64, two waves, four          where 64x64 tiles leave half of the units without work: what a unit requests bounds
//      stages of 64                    them, and these request three quarters of it.  T=512 N=1024 K=4096 forward 16.2 ->
//                                      14.3, gradient 15.1 -> 13.5, K=1024 7.0 -> 6.4; T=512 N=256 K=256 4.8 -> 3.9 (not
//                                      two to a unit: T=1024 N=1024 K=4096 17 -> 21.  Six stages: that gradient 11.9, but
//                                      beside the weight gradients' stream all of a layer's backward 1.5% slower)
//  10: 32x32, one wave, four stages    half of it.  T=256 N=1024 K=4096 14.6 -> 12.8, 14.9 -> 12.3 (32x64: 12.9, 13.1);
//      of 64                           T=256 N=256 K=512 5.7 -> 4.1 (4.4)
//  12: 128x64, four stages of 64,      at most one workgroup for each unit.  T=2048 N=1024 K=4096 forward 25.5 (4) -> 24.0,
//      eight waves                     gradient 24.7 -> 21.1; T=1400 24.5 -> 20.6, 24.1 -> 20.0 (with more tiles than units
//                                      T=2560 39.4 -> 40.9, T=3000 N=768 28.1 -> 31.9).  Beside the weight gradients' stream 96 KB leave
//                                      room for one of its workgroups instead of two halves: 4 layers of 768 with 2048 rows
//                                      1977 us in four waves, 1990 with this tile there, 1951 with tile 4
//      (In four waves beside the weight gradients, 2 layers, a process each: 1024 wide, F = 4096, 1280 rows 542 (4) and 554,
//      F = 2048 446 and 453, 768 wide, 6 x 600 rows 954 and 974, 640 wide 479 and 484; from 1700 rows on 1024 wide 0-1% faster
//      (1904 rows 581 and 577; four micro-batches of 512, F = 4096, 638 and 645), 1088 to 1536 wide 0.6% faster to 1.3% slower,
//      2048 wide 1.6% faster to 0.3% slower.  1024 wide, F = 2048, 2 x 768 rows is 2% faster with them, but not by the
//      product: the chip clocks 2.20 GHz there with the eight waves and 2.31 with four, the kernels that are the same in both
//      included, where 3 x 512 and 1 x 1280 rows have 2.32 with either.)
//      (Which of 4 and 12 forward products take beside the lanes of re-computation, which are not `shared`, is all one: within 0.3%
//      over 40 stages of 3 layers 512 to 1024 wide, 1264 to 5464 rows.)
// (4 and 12, iterations against 4 in four waves: 4 layers of 768 with 600 rows a micro-batch 1875 -> 1831 us, 2 of 1024 with 512 and
// heads of 128 646 -> 640, 3 of 640 with 1024 1334 -> 1312, 2 of 1024 with 510 647 -> 638.)
// A stream restricted to part of the units (GemmArgs::units) moves the lines with it: four stages of 2048 rows on 64
// units each, 36.7 -> 32.2 ms per iteration.  Where another stream's products run beside this one (GemmArgs::shared: the
// data gradients beside the weight gradients) the tile with the whole LDS keeps them off its unit, and the four waves of tile
// 8 get less of a unit than the eight of tile 3 where the weight gradients fill the chip: 12 layers of 1024 with 4096 rows
// take 25.7 ms with tile 6, 24.6 with 8 and 24.3 with 3, 4 of 1536 with 2048 rows 9.19 (8) and 8.97 (3), 4 of 832 with 4096
// rows 7.13 and 7.06.  Tile 8 in narrower layers and for the wide output of few rows: 512 wide, 6144 rows 5.10 and 5.19; 640,
// 5120 rows 6.13 and 6.19; 768, 4096 rows 6.00 and 6.01; 1024 wide, 1024 rows 5.49 and 5.54.
// (The lines between those points -- K >= 2048, N <= 1024, three quarters of the units -- were read off widths of 256,
// 1024 and 2048 and 512 to 8192 rows.)
// K segments that are no multiple of 64 have the 128x128 tile in two stages and the 128x64 one in three, both of eight waves.
// The latter against four waves, 2 layers: 256 wide, F = 1000, 2 x 256 rows 336 and 347, 768 wide, F = 3000, 3 x 600 rows 1016 and
// 1029, 1024 wide, F = 4008, 512 rows 887 and 896, 1536 rows 1208 and 1218; the same with other streams beside it.  (2560 rows
// of 1024 1751 and 1727, F = 2040 1327 and 1318, F = 1000 1106 and 1111; 2600 of 896 1724 and 1727, 3096 1962 and 1956.)
// No bit of a result depends on the choice: an output element is one wave's sum in ascending k whatever the tile.
static int choose_tile(const GemmArgs& g, bool tt, bool short_k) {
  auto tiles = [&](long m, long n) { return ((g.M + m - 1) / m) * ((g.N + n - 1) / n) * g.batch; };
  const long t128 = tiles(128, 128), U = g.units > 0 ? g.units : 256, most = 3 * U / 4;
  const bool bsum = (g.epi & EPI_BSUM) != 0;   // (offered for the weight-gradient layout only)
  int tile = g.tile < 0 || g.tile == 11 || g.tile > 12 ? 7 : g.tile;   // GemmArgs::tile names a configuration instead (tests, timing)
  if (tile == 5 && !tt) tile = 3;
  if (tile == 8 && g.a_kstrided) tile = tt ? 5 : 3;   // (products whose rows are activations only)
  if (tile >= 9 && g.a_kstrided) tile = 7;
  if (bsum && (tile == 1 || tile == 2 || tile == 6)) tile = 0;
  if (short_k) return tile == 3 || (tile != 4 && t128 >= most) ? 3 : 4;
  if (g.epi & EPI_SEGACC) tile = 0;
  if (tile) return tile;
  if (tt) {
    if (t128 >= most) return 5;
    return tiles(128, 64) >= most ? 4 : 7;
  }
  const bool second = (g.epi & (EPI_ADD | EPI_MUL | EPI_GELU)) != 0;   // an epilogue that moves a second matrix
  const long t256 = tiles(256, 128);
  if (tiles(256, 256) >= most && !(g.epi & (EPI_ADD | EPI_AUX32))) return 1;
  if (t256 >= most && t256 <= U && (g.K >= 2048 || !second || g.N <= 1024)) return 2;
  if (t128 > U) return 3;
  // (A k-strided, B k-contiguous has no 8, and is never beside another stream.  Us for tiles 3 / 4 / 6: 2048 x 1920 x 512 8.7 / 9.6 / 8.8,
  // 2048 x 2048 x 1024 11.8 / 13.7 / 12.6, 1536 x 2048 x 1536 18.4 / 16.0 / 13.6)
  if (t128 >= most) {
    if (g.a_kstrided) return g.K > 1024 ? 6 : 3;
    if (g.shared) return g.M >= 8 * U && g.N > 768 ? 3 : 8;
    return g.K >= 2048 ? 6 : 8;
  }
  if (tiles(32, 64) <= U && !g.a_kstrided) return tiles(32, 32) <= U ? 10 : 9;
  if (g.K >= 2048 && tiles(64, 64) > U) return !g.a_kstrided && !g.shared && tiles(128, 64) <= U ? 12 : 4;
  return 7;
}

GemmArgs wgrad_args(const WgradGroup& w, int i) {
  const WgradProblem& p = w.p[i];
  GemmArgs g{};
  g.A = p.A; g.B = p.B; g.C = p.C; g.M = g.m_valid = p.M; g.N = g.n_valid = p.N; g.K = g.k_valid = w.K;
  g.lda = p.lda; g.ldb = p.ldb; g.ldc = p.ldc; g.a_kstrided = g.b_kstrided = 1; g.batch = 1;
  g.kseg_len = w.kseg; g.segA = (long)w.kseg * p.lda; g.segB = (long)w.kseg * p.ldb;
  g.epi = EPI_ACC32 | (p.bsum ? EPI_BSUM : 0) | (w.K > w.kseg ? EPI_SEGACC : 0);
  g.bsum = p.bsum; g.units = w.units;
  return g;
}

bool wgrad_group_takes(Dtype dt, const WgradGroup& w) {
  if (w.n < 1 || w.n > WgradGroup::MAX || w.kseg < 1 || w.K < w.kseg || w.K % w.kseg) return false;
  for (int i = 0; i < w.n; ++i) {
    const GemmArgs g = wgrad_args(w, i);
    if (!(dt == DT_BF16 ? gemm_uses_mfma(dt, g) : gemm_f32_takes(g))) return false;
  }
  return true;
}

hipError_t launch_wgrad_group(Dtype dt, const WgradGroup& w, hipStream_t st) {
  return dt == DT_BF16 ? launch_wgrad_group_mfma(w, st) : launch_wgrad_group_f32(w, st);
}

hipError_t launch_gemm(Dtype dt, const GemmArgs& g, hipStream_t st, GemmPlan* plan) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
  const bool mfma = gemm_uses_mfma(dt, g);
  if ((g.epi & EPI_ROWDOT) && !mfma) return hipErrorInvalidValue;  // only the MFMA kernel's epilogue has it
  if (mfma) {
    const bool tt = g.a_kstrided && g.b_kstrided;   // the weight-gradient layout
    const bool short_k = g.kseg_len % 64 != 0 && !tt;
    const int tile = choose_tile(g, tt, short_k);
    const GemmLaunch l{tile, short_k, st, plan};
    if (tt) return launch_mfma_tt(g, l);
    if (g.a_kstrided) return launch_mfma_tn(g, l);
    return g.b_kstrided ? launch_mfma_nt(g, l) : launch_mfma_nn(g, l);
  }
  if (plan) return hipErrorInvalidValue;
  if (dt == DT_F32 && gemm_f32_takes(g)) return launch_gemm_f32(g, st);
  dim3 blk(32, 8);
  dim3 grid((g.N + 31) / 32, (g.M + 7) / 8, g.batch);
  if (dt == DT_BF16)
    hipLaunchKernelGGL(gemm_plain_kernel<bf16>, grid, blk, 0, st, g);
  else
    hipLaunchKernelGGL(gemm_plain_kernel<float>, grid, blk, 0, st, g);
  return hipGetLastError();
}

}  // namespace dapple
