// Self-attention of an fp32 stage on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32): the formulas and the
// orientation of attention.hip -- a wave owns 16 query rows (forward, dq) or 16 key rows (dk/dv), 32-row blocks of the
// other side stream through LDS, the accumulator's lane index is the row the wave owns, so the probabilities leave
// the first product in the layout the second one takes.  A 16x16x4 instruction takes one fp32 per lane and operand,
// so no permutation and no transpose read is needed.
//
// What bounds it: the matrix pipe at the fp32 rate (32 clocks per 2048 flops), LDS a quarter of that; the smallest
// wave tile (16 rows) is taken because it reaches the most SIMDs (b = 2, s = 512, 16 heads of 64: 1024 waves, one per
// SIMD; 32-row tiles would leave half of them idle) and, on the smallest stages, has the shortest chain.
// delta = rowsum(dctx o ctx) is computed where it is used: by the dq waves from the rows they own, by the dk/dv
// workgroups while they load a query block; a kernel of its own would cost a launch and save nothing.
// b = 4, s = 512, 16 heads of 64 (two micro-batches in a stage): 54 us forward, 142 us backward (79 and 61 TFLOP/s of
// useful work); the library's exp2f, which keeps denormal probabilities, is 3% of that.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace dapple {

static constexpr float LOG2E = 1.4426950408889634f;

#define MFMA4(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0)

// D: the head block's width (16, 32, 64 or 128; narrower heads are padded with zeros); blocks of 32 rows
constexpr int BR = 32;
template <int D>
struct F32Block {
  // row stride D + 8 floats: the four lane groups of a 4-byte read lie 4 rows = 32 banks (mod 64) apart
  static constexpr int LD = D + 8, CPR = D / 4, N = BR * CPR / 256 > 0 ? BR * CPR / 256 : 1;
  f32x4 c[N];
  __device__ __forceinline__ void load(const float* g, int ldg, int tid, int rows, int d) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int p = tid + 256 * i, r = p / CPR, k = p % CPR * 4;
      c[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (p < BR * CPR && r < rows && k < d) c[i] = *(const f32x4*)(g + (long)r * ldg + k);
    }
  }
  __device__ __forceinline__ void store(float* S, int tid) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int p = tid + 256 * i;
      if (p < BR * CPR) *(f32x4*)(S + p / CPR * LD + p % CPR * 4) = c[i];
    }
  }
};
// row r0 + (lane & 15), k = 16 kk + 4 (lane >> 4) + 0..3
template <int D>
__device__ __forceinline__ f32x4 frow(const float* S, int r0, int kk, int lane) {
  return *(const f32x4*)(S + (r0 + (lane & 15)) * (D + 8) + 16 * kk + 4 * (lane >> 4));
}
// column c0 + (lane & 15) of row r0 + 4 (lane >> 4) + e
template <int D>
__device__ __forceinline__ float fcol(const float* S, int c0, int r0, int e, int lane) {
  return S[(r0 + 4 * (lane >> 4) + e) * (D + 8) + c0 + (lane & 15)];
}
// the row a lane owns in registers, k = 16 kk + 4 (lane >> 4) + 0..3
template <int D>
__device__ __forceinline__ void own_row(const float* row, bool ok, int d, int lane, f32x4 (&f)[D / 16]) {
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    const int k = 16 * kk + 4 * (lane >> 4);
    f[kk] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (ok && k < d) f[kk] = *(const f32x4*)(row + k);
  }
}
__device__ __forceinline__ float over_groups_sum(float v) {   // the four lanes of one owned row, pairs first
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

template <int D>
__global__ __launch_bounds__(256) void attn_fwd_f32(AttnArgs a, float scale2) {
  constexpr int NK = D / 16;
  __shared__ __attribute__((aligned(16))) float Ks[BR * (D + 8)];
  __shared__ __attribute__((aligned(16))) float Vs[BR * (D + 8)];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g4 = lane >> 4;
  const int bi = (a.head0 + blockIdx.y) / a.A, hh = (a.head0 + blockIdx.y) % a.A;
  const long hb = (long)bi * a.s * a.H + hh * a.d;
  const float *Q = (const float*)a.q + hb, *K = (const float*)a.k + hb, *V = (const float*)a.v + hb;
  const int qrow = blockIdx.x * 64 + wave * 16 + (lane & 15);
  const bool qok = qrow < a.s;
  f32x4 qf[NK];
  own_row<D>(Q + (long)qrow * a.H, qok, a.d, lane, qf);
  F32Block<D> kb, vb;
  kb.load(K, a.H, tid, a.s, a.d);
  vb.load(V, a.H, tid, a.s, a.d);
  float m = -INFINITY, l = 0.f;
  f32x4 o[NK];   // rows d = 16 i + 4 g4 + e, column = the lane's query
#pragma unroll
  for (int i = 0; i < NK; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < a.s; k0 += BR) {
    __syncthreads();
    kb.store(Ks, tid);
    vb.store(Vs, tid);
    __syncthreads();
    if (k0 + BR < a.s) {
      kb.load(K + (long)(k0 + BR) * a.H, a.H, tid, a.s - k0 - BR, a.d);
      vb.load(V + (long)(k0 + BR) * a.H, a.H, tid, a.s - k0 - BR, a.d);
    }
    f32x4 p[2];
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t) {   // rows: key k0 + 16 t + 4 g4 + e, column: query
      f32x4 s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        const f32x4 kf = frow<D>(Ks, 16 * t, kk, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) s = MFMA4(kf[e], qf[kk][e], s);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[t][e] = k0 + 16 * t + 4 * g4 + e < a.s ? s[e] * scale2 : -INFINITY;
        mx = fmaxf(mx, p[t][e]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mn = fmaxf(m, mx), alpha = exp2f(m - mn);
    float rs = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[t][e] = exp2f(p[t][e] - mn);
        rs += p[t][e];
      }
    l = l * alpha + over_groups_sum(rs);
    m = mn;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {
#pragma unroll
      for (int i = 0; i < NK; ++i) o[i] *= alpha;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < NK; ++i) o[i] = MFMA4(fcol<D>(Vs, 16 * i, 16 * t, e, lane), p[t][e], o[i]);
  }
  if (qok) {
    const float inv = 1.0f / l;
    float* C = (float*)a.ctx + hb + (long)qrow * a.H;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int col = 16 * i + 4 * g4;
      if (col < a.d) *(f32x4*)(C + col) = o[i] * inv;
    }
    if (g4 == 0) a.lse[((long)bi * a.A + hh) * a.s + qrow] = m + log2f(l);
  }
}

template <int D>
__device__ __forceinline__ void dq_f32(const AttnArgs& a, float scale2, float scale, float* Ks, float* Vs) {
  constexpr int NK = D / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g4 = lane >> 4;
  const int bi = (a.head0 + blockIdx.y) / a.A, hh = (a.head0 + blockIdx.y) % a.A;
  const long hb = (long)bi * a.s * a.H + hh * a.d;
  const float *K = (const float*)a.k + hb, *V = (const float*)a.v + hb;
  const int qrow = blockIdx.x * 64 + wave * 16 + (lane & 15);
  const bool qok = qrow < a.s;
  const long ro = hb + (long)qrow * a.H;
  f32x4 qf[NK], gf[NK];
  own_row<D>((const float*)a.q + ro, qok, a.d, lane, qf);
  own_row<D>((const float*)a.dctx + ro, qok, a.d, lane, gf);
  const float Lq = qok ? a.lse[((long)bi * a.A + hh) * a.s + qrow] : 0.f;
  float Dq = 0.f;
  {
    f32x4 cf[NK];
    own_row<D>((const float*)a.ctx + ro, qok, a.d, lane, cf);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e) Dq = fmaf(cf[kk][e], gf[kk][e], Dq);
    Dq = over_groups_sum(Dq);
  }
  f32x4 dq[NK];
#pragma unroll
  for (int i = 0; i < NK; ++i) dq[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  F32Block<D> kb, vb;
  kb.load(K, a.H, tid, a.s, a.d);
  vb.load(V, a.H, tid, a.s, a.d);
  for (int k0 = 0; k0 < a.s; k0 += BR) {
    __syncthreads();
    kb.store(Ks, tid);
    vb.store(Vs, tid);
    __syncthreads();
    if (k0 + BR < a.s) {
      kb.load(K + (long)(k0 + BR) * a.H, a.H, tid, a.s - k0 - BR, a.d);
      vb.load(V + (long)(k0 + BR) * a.H, a.H, tid, a.s - k0 - BR, a.d);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      f32x4 s{0.f, 0.f, 0.f, 0.f}, dp{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        const f32x4 kf = frow<D>(Ks, 16 * t, kk, lane), vf = frow<D>(Vs, 16 * t, kk, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s = MFMA4(kf[e], qf[kk][e], s);
          dp = MFMA4(vf[e], gf[kk][e], dp);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float ds = exp2f(s[e] * scale2 - Lq) * (dp[e] - Dq);
        if (k0 + 16 * t + 4 * g4 + e >= a.s) ds = 0.f;
#pragma unroll
        for (int i = 0; i < NK; ++i) dq[i] = MFMA4(fcol<D>(Ks, 16 * i, 16 * t, e, lane), ds, dq[i]);
      }
    }
  }
  if (qok) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int col = 16 * i + 4 * g4;
      if (col < a.d) *(f32x4*)((float*)a.dq + ro + col) = dq[i] * scale;
    }
  }
}

template <int D>
__device__ __forceinline__ void dkdv_f32(const AttnArgs& a, float scale2, float scale, float* Qs, float* Gs, float* Ls,
                                         float* Ds) {
  constexpr int NK = D / 16;
  typedef F32Block<D> Blk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g4 = lane >> 4;
  const int bi = (a.head0 + blockIdx.y) / a.A, hh = (a.head0 + blockIdx.y) % a.A;
  const long hb = (long)bi * a.s * a.H + hh * a.d;
  const float *Q = (const float*)a.q + hb, *G = (const float*)a.dctx + hb, *O = (const float*)a.ctx + hb;
  const float* lse = a.lse + ((long)bi * a.A + hh) * a.s;
  const int krow = blockIdx.x * 64 + wave * 16 + (lane & 15);
  const bool kok = krow < a.s;
  const long ro = hb + (long)krow * a.H;
  f32x4 kf[NK], vf[NK], dk[NK], dv[NK];
  own_row<D>((const float*)a.k + ro, kok, a.d, lane, kf);
  own_row<D>((const float*)a.v + ro, kok, a.d, lane, vf);
#pragma unroll
  for (int i = 0; i < NK; ++i) dk[i] = dv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  Blk qb, gb, ob;
  float L = 0.f;
  auto load = [&](int q0) {
    qb.load(Q + (long)q0 * a.H, a.H, tid, a.s - q0, a.d);
    gb.load(G + (long)q0 * a.H, a.H, tid, a.s - q0, a.d);
    ob.load(O + (long)q0 * a.H, a.H, tid, a.s - q0, a.d);
    L = tid < BR && q0 + tid < a.s ? lse[q0 + tid] : 0.f;
  };
  load(0);
  for (int q0 = 0; q0 < a.s; q0 += BR) {
    __syncthreads();
    qb.store(Qs, tid);
    gb.store(Gs, tid);
    if (tid < BR) Ls[tid] = L;
    // a row's CPR chunks lie in CPR consecutive lanes of one wave
#pragma unroll
    for (int i = 0; i < Blk::N; ++i) {
      float t = (gb.c[i][0] * ob.c[i][0] + gb.c[i][1] * ob.c[i][1]) + (gb.c[i][2] * ob.c[i][2] + gb.c[i][3] * ob.c[i][3]);
#pragma unroll
      for (int x = 1; x < Blk::CPR; x <<= 1) t += __shfl_xor(t, x, 64);
      const int p = tid + 256 * i;
      if (p < BR * Blk::CPR && p % Blk::CPR == 0) Ds[p / Blk::CPR] = t;
    }
    __syncthreads();
    if (q0 + BR < a.s) load(q0 + BR);
#pragma unroll
    for (int t = 0; t < 2; ++t) {   // rows: query q0 + 16 t + 4 g4 + e, column: key
      f32x4 s{0.f, 0.f, 0.f, 0.f}, dp{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        const f32x4 qf = frow<D>(Qs, 16 * t, kk, lane), gf = frow<D>(Gs, 16 * t, kk, lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s = MFMA4(qf[e], kf[kk][e], s);
          dp = MFMA4(gf[e], vf[kk][e], dp);
        }
      }
      const f32x4 L4 = *(const f32x4*)(Ls + 16 * t + 4 * g4), D4 = *(const f32x4*)(Ds + 16 * t + 4 * g4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // a query beyond the last: zero rows, lse 0, delta 0 -- probability 1 times a zero row, dS = 0
        const float p = exp2f(s[e] * scale2 - L4[e]), ds = p * (dp[e] - D4[e]);
#pragma unroll
        for (int i = 0; i < NK; ++i) {
          dv[i] = MFMA4(fcol<D>(Gs, 16 * i, 16 * t, e, lane), p, dv[i]);
          dk[i] = MFMA4(fcol<D>(Qs, 16 * i, 16 * t, e, lane), ds, dk[i]);
        }
      }
    }
  }
  if (kok) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int col = 16 * i + 4 * g4;
      if (col < a.d) {
        *(f32x4*)((float*)a.dk + ro + col) = dk[i] * scale;
        *(f32x4*)((float*)a.dv + ro + col) = dv[i];
      }
    }
  }
}

// grid.z = 0: dq, 1: dk and dv
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_f32(AttnArgs a, float scale2, float scale) {
  __shared__ __attribute__((aligned(16))) float X[BR * (D + 8)];
  __shared__ __attribute__((aligned(16))) float Y[BR * (D + 8)];
  __shared__ __attribute__((aligned(16))) float Ls[BR];
  __shared__ __attribute__((aligned(16))) float Ds[BR];
  if (blockIdx.z == 0) dq_f32<D>(a, scale2, scale, X, Y);
  else dkdv_f32<D>(a, scale2, scale, X, Y, Ls, Ds);
}

// ------------------------------------------------------------------ launchers
static bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

bool attn_f32_takes(const AttnArgs& a) {
  return a.d % 4 == 0 && a.d <= 128 && a.H % 4 == 0 && al16(a.q) && al16(a.k) && al16(a.v) && al16(a.ctx) &&
         (a.dctx == nullptr || (al16(a.dctx) && al16(a.dq) && al16(a.dk) && al16(a.dv)));
}

template <typename F>
static void pick_width(int d, F&& f) {
  if (d <= 16) f(std::integral_constant<int, 16>{});
  else if (d <= 32) f(std::integral_constant<int, 32>{});
  else if (d <= 64) f(std::integral_constant<int, 64>{});
  else f(std::integral_constant<int, 128>{});
}

hipError_t launch_attn_fwd_f32(const AttnArgs& a, hipStream_t st) {
  const float scale2 = LOG2E / sqrtf((float)a.d);
  return attn_launches(a, [&](const AttnArgs& l, int heads) {
    const dim3 grid((a.s + 63) / 64, heads);
    pick_width(a.d, [&](auto D) { hipLaunchKernelGGL(attn_fwd_f32<decltype(D)::value>, grid, dim3(256), 0, st, l, scale2); });
    return hipGetLastError();
  });
}

hipError_t launch_attn_bwd_f32(const AttnArgs& a, hipStream_t st) {
  const float scale = 1.0f / sqrtf((float)a.d), scale2 = LOG2E * scale;
  return attn_launches(a, [&](const AttnArgs& l, int heads) {
    const dim3 grid((a.s + 63) / 64, heads, 2);
    pick_width(a.d, [&](auto D) { hipLaunchKernelGGL(attn_bwd_f32<decltype(D)::value>, grid, dim3(256), 0, st, l, scale2, scale); });
    return hipGetLastError();
  });
}

}  // namespace dapple
