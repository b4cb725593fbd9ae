// What the GEMM kernels share: which tile a workgroup computes, and the epilogue of one output element (or four).
#pragma once
#include "device_common.h"
#include "kernels.h"

namespace dapple {

// Tile index.  Consecutive workgroups land on different XCDs (round-robin over 8), and
// each XCD has its own L2.  Cut the tile grid into pm x pn = 8 rectangles, one per XCD,
// so that the A and B panels an XCD touches are as few as possible and are reused by
// all its tiles out of its L2; inside a rectangle walk down its columns of tiles.
__device__ __forceinline__ void tile_of(int bid, int tiles_m, int tiles_n, int BM, int BN, int& tm, int& tn) {
  const int ntiles = tiles_m * tiles_n;
  int pm = 0, best = 1 << 30;
#pragma unroll
  for (int c = 1; c <= 8; c <<= 1) {
    int pn = 8 / c;
    if (tiles_m % c == 0 && tiles_n % pn == 0) {
      int cost = (tiles_m / c) * BM + (tiles_n / pn) * BN;
      if (cost < best) { best = cost; pm = c; }
    }
  }
  if (pm == 0 || (ntiles & 7)) {
    tm = bid / tiles_n;
    tn = bid % tiles_n;
  } else {
    const int pn = 8 / pm, rm = tiles_m / pm, rn = tiles_n / pn;
    const int xcd = bid & 7, local = bid >> 3;
    const int lm = local % rm, ln = local / rm;
    tm = (xcd / pn) * rm + lm;
    tn = (xcd % pn) * rn + ln;
  }
}

template <typename T>
__device__ __forceinline__ void epilogue_store(const GemmArgs& g, long zc, long zbias, int row, int col, float t) {
  if (g.epi & EPI_BIAS) t += to_f32(((const T*)g.bias)[zbias + col]);
  if (g.epi & (EPI_ADD | EPI_MUL)) {
    long ao = zc + (long)row * g.ldaux + col;
    float x = (g.epi & EPI_AUX32) ? ((const float*)g.aux)[ao] : to_f32(((const T*)g.aux)[ao]);
    if (g.epi & EPI_AUXLN)
      x = (x - g.ln_stats[2 * row]) * g.ln_stats[2 * row + 1] * to_f32(((const T*)g.ln_gamma)[col]) + to_f32(((const T*)g.ln_beta)[col]);
    t = (g.epi & EPI_ADD) ? t + x : t * x;
  }
  long o = zc + (long)row * g.ldc + col;
  if (g.epi & EPI_GELU) {
    float a, b;
    gelu_both(t, a, b);
    ((T*)g.C)[o] = from_f32<T>(a);
    ((T*)g.C2)[o] = from_f32<T>(b);
  } else if (g.epi & EPI_ACC32) {
    ((float*)g.C)[o] += t;
  } else if (g.epi & EPI_OUT32) {
    ((float*)g.C)[o] = t;
  } else {
    ((T*)g.C)[o] = from_f32<T>(t);
  }
}

// four consecutive columns of one row of an fp32 product (every pointer and stride 16-byte aligned): what the epilogue
// reads, and the store
struct Epilogue4 {
  f32x4 bias, x, c;
};
__device__ __forceinline__ Epilogue4 epilogue_load4(const GemmArgs& g, long zc, long zbias, int row, int col) {
  Epilogue4 in{};
  if (g.epi & EPI_BIAS) in.bias = *(const f32x4*)((const float*)g.bias + zbias + col);
  if (g.epi & (EPI_ADD | EPI_MUL)) in.x = *(const f32x4*)((const float*)g.aux + zc + (long)row * g.ldaux + col);
  if (g.epi & EPI_ACC32) in.c = *(const f32x4*)((const float*)g.C + zc + (long)row * g.ldc + col);
  return in;
}
__device__ __forceinline__ void epilogue_store4(const GemmArgs& g, long zc, int row, int col, f32x4 t, const Epilogue4& in) {
  if (g.epi & EPI_BIAS) t += in.bias;
  if (g.epi & (EPI_ADD | EPI_MUL)) t = (g.epi & EPI_ADD) ? t + in.x : t * in.x;
  float* const c = (float*)g.C + zc + (long)row * g.ldc + col;
  if (g.epi & EPI_GELU) {
    f32x4 a, b;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x, y;
      gelu_both(t[e], x, y);
      a[e] = x;
      b[e] = y;
    }
    *(f32x4*)c = a;
    *(f32x4*)((float*)g.C2 + zc + (long)row * g.ldc + col) = b;
  } else if (g.epi & EPI_ACC32) {
    *(f32x4*)c = in.c + t;
  } else {
    *(f32x4*)c = t;
  }
}

}  // namespace dapple
