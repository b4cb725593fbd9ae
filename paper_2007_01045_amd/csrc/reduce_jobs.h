// One workgroup's part of a ReduceJob (kernels.h): 64 columns.
#pragma once
#include "kernels.h"

namespace dapple {

// The summation of a job is that of partial_reduce_kernel, addition for addition, and with several micro-batches each
// one's sum is added to the output on its own, in order.  Four waves per micro-batch, ngrp micro-batches at a time (256
// ngrp threads); red: 4 ngrp rows of LDS.  Every thread of the workgroup calls it, with the same job.
__device__ __forceinline__ void reduce_columns(const ReduceJob& job, int nmb, long mb_stride, int block, int ngrp, float (*red)[64]) {
  const int lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3, grp = threadIdx.x >> 8;
  const int c = block * 64 + lane;
  if (block * 64 >= job.cols) return;   // the whole workgroup: no barrier is skipped by part of it
  for (int i0 = 0; i0 < nmb; i0 += ngrp) {
    float t = 0.f;
    if (c < job.cols && i0 + grp < nmb) {
      const float* p = job.partial + (i0 + grp) * mb_stride + c;
      const long stride = job.stride;
      const int nblk = job.nblk;
      int b = w;
      // 32 loads in flight per wave: the launch is a hundred workgroups waiting for memory
      for (; b + 124 < nblk; b += 128) {
        float x[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) x[u] = p[(long)(b + 4 * u) * stride];
#pragma unroll
        for (int u = 0; u < 32; ++u) t += x[u];
      }
      for (; b + 28 < nblk; b += 32) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[(long)(b + 4 * u) * stride];
#pragma unroll
        for (int u = 0; u < 8; ++u) t += x[u];
      }
      for (; b < nblk; b += 4) t += p[(long)b * stride];
    }
    red[grp * 4 + w][lane] = t;
    __syncthreads();
    if (threadIdx.x < 64 && c < job.cols) {
      float o = job.out[c];
      for (int q = 0; q < ngrp && i0 + q < nmb; ++q) {
        float r = red[4 * q][lane] + red[4 * q + 1][lane];
        r += red[4 * q + 2][lane];
        r += red[4 * q + 3][lane];
        o += r;
      }
      job.out[c] = o;
    }
    __syncthreads();
  }
}

}  // namespace dapple
