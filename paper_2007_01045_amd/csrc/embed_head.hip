// Kernels of the two optional ends of a stage.
//
// First stage (embedding block):  x = LN(E_w[id] + E_p[pos]),  pos = row % s.
//   forward : embed_gather writes e = E_w[id] + E_p[pos] (the LayerNorm kernels do the rest)
//   backward: dE_w[id] += sum of de over the rows that carry this id, added in ascending row
//             order by one wave per id (no atomics: reproducible bit for bit);
//             dE_p[pos] += sum over the sequences of the micro-batch, ascending.
//
// Last stage (masked-LM head):  the rows whose target is >= 0 are gathered (ascending) into a
//   dense block r, t = LN(GELU(r Wt + bt)), z = t E_out^T + b_out,
//   loss = loss_scale * sum_rows (logsumexp(z) - z[target]),  dz = loss_scale * (softmax(z) - onehot).
//   The products are GEMM launches; here are the compaction, the gather / scatter of rows, the
//   row-wise cross-entropy and an element-wise product.
#include "device_common.h"
#include "kernels.h"

namespace dapple {

// ------------------------------------------------------------------ embedding
template <typename T>
__global__ void embed_gather_kernel(const int32_t* __restrict__ ids, const T* __restrict__ Ew,
                                    const T* __restrict__ Ep, T* __restrict__ e, int rows, int s, int H, int vocab) {
  int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  int id = ids[row];
  id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);  // ids outside the table are clamped, never dereferenced
  const T* a = Ew + (long)id * H;
  const T* b = Ep + (long)(row % s) * H;
  for (int c = lane; c < H; c += 64) e[(long)row * H + c] = from_f32<T>(to_f32(a[c]) + to_f32(b[c]));
}

// One wave per row r of the nmb micro-batches: if r is the first row of them all with its id, it owns the id's row of
// the table and adds, micro-batch after micro-batch, the sum of that micro-batch's rows with this id in ascending
// order.  The ids are scanned once (a lane holds NCH * V columns of the sum in registers); scanning them again for every
// 64 columns took 72 us for 1024 rows of 1024 columns.
template <typename T, int NCH>
__global__ __launch_bounds__(256) void embed_scatter_kernel(const int32_t* __restrict__ ids, const T* __restrict__ de,
                                                            float* __restrict__ dEw, int rows, int nmb, int H, int vocab) {
  constexpr int V = 16 / sizeof(T);
  typedef T TV __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x & 63, r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows * nmb) return;
  auto id_at = [&](int q) {   // ids outside the table are clamped, as in the forward
    const int v = ids[q];
    return v < 0 ? 0 : (v >= vocab ? vocab - 1 : v);
  };
  const int id = id_at(r);
  for (int base = 0; base < r; base += 256) {   // an earlier row with the same id owns the sum
    bool hit = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = base + 64 * u + lane;
      hit = hit || (q < r && id_at(q) == id);
    }
    if (__ballot(hit)) return;
  }
  float acc[NCH][V], tot[NCH][V];
  auto add_row = [&](int q) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int col = (c * 64 + lane) * V;
      if (col < H) {
        const TV x = *(const TV*)(de + (long)q * H + col);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[c][e] += to_f32((T)x[e]);
      }
    }
  };
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (c * 64 + lane) * V;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      tot[c][e] = col < H ? dEw[(long)id * H + col + e] : 0.f;
      acc[c][e] = 0.f;
    }
  }
  for (int mb = r / rows; mb < nmb; ++mb) {
    const int end = (mb + 1) * rows;
    bool any = false;
    for (int base = max(r, mb * rows); base < end; base += 256) {
      unsigned long long m[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = base + 64 * u + lane;
        m[u] = __ballot(q < end && id_at(q < end ? q : r) == id);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        while (m[u]) {  // ascending rows
          const int j = __builtin_ctzll(m[u]);
          m[u] &= m[u] - 1;
          add_row(base + 64 * u + j);
          any = true;
        }
    }
    if (any) {
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int e = 0; e < V; ++e) {
          tot[c][e] += acc[c][e];
          acc[c][e] = 0.f;
        }
    }
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int col = (c * 64 + lane) * V;
    if (col < H)
#pragma unroll
      for (int e = 0; e < V; ++e) dEw[(long)id * H + col + e] = tot[c][e];
  }
}

template <typename T>
__global__ void embed_pos_grad_kernel(const T* __restrict__ de, float* __restrict__ dEp, int b, int s, int H, int nmb) {
  long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)s * H) return;
  float tot = dEp[idx];
  for (int mb = 0; mb < nmb; ++mb) {
    float acc = 0.f;
    for (int bi = 0; bi < b; ++bi) acc += to_f32(de[(long)(mb * b + bi) * s * H + idx]);
    tot += acc;
  }
  dEp[idx] = tot;
}

// ------------------------------------------------------------------ masked-LM head
// rows_idx[i], i < np: i-th row (ascending) whose target is >= 0, -1 beyond the count; tgt[i] its
// target (clamped into the vocabulary).  info[0] = count, info[1] = 1 if more than cap rows
// are predicted (the surplus is dropped and the stage reports the overflow at the next sync).
__global__ __launch_bounds__(1024) void mlm_compact_kernel(const int32_t* __restrict__ targets, int T, int cap,
                                                           int np, int vocab, int32_t* __restrict__ rows_idx,
                                                           int32_t* __restrict__ tgt, int32_t* __restrict__ info) {
  __shared__ int wave_cnt[16];
  __shared__ int running;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  targets += (long)blockIdx.x * T;   // micro-batch blockIdx.x
  rows_idx += (long)blockIdx.x * np;
  tgt += (long)blockIdx.x * np;
  if (tid == 0) running = 0;
  for (int i = tid; i < np; i += 1024) {  // all np >= cap entries, padding rows included
    rows_idx[i] = -1;
    tgt[i] = 0;
  }
  __syncthreads();
  for (int base = 0; base < T; base += 1024) {
    int r = base + tid;
    bool on = r < T && targets[r] >= 0;
    unsigned long long m = __ballot(on);
    if (lane == 0) wave_cnt[wave] = __builtin_popcountll(m);
    __syncthreads();
    int before = running;
    for (int w = 0; w < wave; ++w) before += wave_cnt[w];
    int pos = before + __builtin_popcountll(m & ((1ull << lane) - 1ull));
    if (on && pos < cap) {
      int t = targets[r];
      rows_idx[pos] = r;
      tgt[pos] = t >= vocab ? vocab - 1 : t;
    }
    __syncthreads();
    if (tid == 0) {
      int tot = 0;
      for (int w = 0; w < 16; ++w) tot += wave_cnt[w];
      running += tot;
    }
    __syncthreads();
  }
  if (tid == 0) {
    info[0] = running < cap ? running : cap;
    if (running > cap) info[1] = 1;
  }
}

// dst[i] = idx[i] >= 0 ? src[idx[i]] : 0   (rows of n16 16-byte pieces; micro-batch blockIdx.y)
__global__ void gather_rows_kernel(const uint4* __restrict__ src, const int32_t* __restrict__ idx, uint4* __restrict__ dst,
                                   int n, int n16, int nsrc) {
  int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n) return;
  const long mb = blockIdx.y;
  const int r = idx[mb * n + i];
  const bool ok = r >= 0 && r < nsrc;
  const uint4* s = src + (mb * nsrc + (ok ? r : 0)) * n16;
  uint4* d = dst + (mb * n + i) * n16;
  for (int c = lane; c < n16; c += 64) d[c] = ok ? s[c] : make_uint4(0, 0, 0, 0);
}
// dst[idx[i]] = src[i] for idx[i] >= 0  (dst zeroed beforehand; the indices are distinct)
__global__ void scatter_rows_kernel(const uint4* __restrict__ src, const int32_t* __restrict__ idx, uint4* __restrict__ dst,
                                    int n, int n16, int ndst) {
  int lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n) return;
  const long mb = blockIdx.y;
  const int r = idx[mb * n + i];
  if (r < 0 || r >= ndst) return;
  for (int c = lane; c < n16; c += 64) dst[(mb * ndst + r) * n16 + c] = src[(mb * n + i) * n16 + c];
}

// one workgroup per gathered row: z = logits + bias over v < V; row_loss = logsumexp(z) - z[tgt];
// dz = loss_scale * (softmax(z) - onehot), zero in the padding columns and in padding rows
template <typename T>
__global__ __launch_bounds__(256) void mlm_ce_kernel(const float* __restrict__ logits, const T* __restrict__ bias,
                                                     const int32_t* __restrict__ rows_idx,
                                                     const int32_t* __restrict__ tgt, int V, int VP, float loss_scale,
                                                     T* __restrict__ dz, float* __restrict__ row_loss) {
  __shared__ float red[4];
  const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* z = logits + (long)i * VP;
  T* d = dz + (long)i * VP;
  if (rows_idx[i] < 0) {
    for (int v = tid; v < VP; v += 256) d[v] = from_f32<T>(0.f);
    if (tid == 0) row_loss[i] = 0.f;
    return;
  }
  float mx = -INFINITY;
  for (int v = tid; v < V; v += 256) mx = fmaxf(mx, z[v] + to_f32(bias[v]));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float sum = 0.f;
  for (int v = tid; v < V; v += 256) sum += __expf(z[v] + to_f32(bias[v]) - mx);
  sum = wave_sum(sum);
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  sum = ((red[0] + red[1]) + red[2]) + red[3];
  const float lse = mx + __logf(sum);
  int t = tgt[i];
  t = t < 0 ? 0 : (t >= V ? V - 1 : t);
  const float inv = 1.0f / sum;
  for (int v = tid; v < VP; v += 256) {
    float g = 0.f;
    if (v < V) {
      g = __expf(z[v] + to_f32(bias[v]) - mx) * inv;
      if (v == t) g -= 1.0f;
      g *= loss_scale;
    }
    d[v] = from_f32<T>(g);
  }
  if (tid == 0) row_loss[i] = lse - (z[t] + to_f32(bias[t]));
}

// The same for vocabularies of up to 4096 NV words with the row's logits in registers: one pass over them instead of
// three (384 rows of 30522 words: 113 us with three passes of 256 threads, 20 with this)
template <typename T, int NV>
__global__ __launch_bounds__(1024) void mlm_ce_regs_kernel(const float* __restrict__ logits, const T* __restrict__ bias,
                                                           const int32_t* __restrict__ rows_idx,
                                                           const int32_t* __restrict__ tgt, int V, int VP, float loss_scale,
                                                           T* __restrict__ dz, float* __restrict__ row_loss) {
  typedef T T4 __attribute__((ext_vector_type(4)));
  __shared__ float red[16];
  __shared__ float ztgt;
  const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* z = logits + (long)i * VP;
  T* d = dz + (long)i * VP;
  const bool live = rows_idx[i] >= 0;
  if (!live) {
    const T4 zero = {from_f32<T>(0.f), from_f32<T>(0.f), from_f32<T>(0.f), from_f32<T>(0.f)};
    for (int v = tid * 4; v < VP; v += 4096) *(T4*)(d + v) = zero;
    if (tid == 0) row_loss[i] = 0.f;
    return;
  }
  int t = tgt[i];
  t = t < 0 ? 0 : (t >= V ? V - 1 : t);
  f32x4 x[NV];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int v = (u * 1024 + tid) * 4;
    x[u] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (v < VP) x[u] = *(const f32x4*)(z + v);   // VP is a multiple of 64
  }
#pragma unroll
  for (int u = 0; u < NV; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int v = (u * 1024 + tid) * 4 + e;
      x[u][e] = v < V ? x[u][e] + to_f32(bias[v]) : -INFINITY;
      if (v == t) ztgt = x[u][e];
      mx = fmaxf(mx, x[u][e]);
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 16; ++w) mx = fmaxf(mx, red[w]);
  __syncthreads();
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < NV; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[u][e] = __expf(x[u][e] - mx);
      sum += x[u][e];
    }
  sum = wave_sum(sum);
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  sum = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) sum += red[w];
  const float inv = 1.0f / sum;
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int v = (u * 1024 + tid) * 4;
    if (v >= VP) continue;
    T4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float g = x[u][e] * inv;
      if (v + e == t) g -= 1.0f;
      o[e] = from_f32<T>(v + e < V ? g * loss_scale : 0.f);
    }
    *(T4*)(d + v) = o;
  }
  if (tid == 0) row_loss[i] = mx + __logf(sum) - ztgt;
}

// out[i] = scale * (sum of micro-batch i's n row losses), in a fixed order: every lane's rows ascending, then the lanes
__global__ __launch_bounds__(64) void loss_sum_kernel(const float* __restrict__ row_loss, int n, float scale, float* __restrict__ out) {
  const float* p = row_loss + (long)blockIdx.x * n;
  float t = 0.f;
  for (int i = threadIdx.x; i < n; i += 64) t += p[i];
  t = wave_sum(t);
  if (threadIdx.x == 0) out[blockIdx.x] = t * scale;
}

template <typename T>
__global__ void mul_kernel(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ c, long n) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) c[i] = from_f32<T>(to_f32(a[i]) * to_f32(b[i]));
}

// ------------------------------------------------------------------ launchers
hipError_t launch_embed_gather(Dtype dt, const int32_t* ids, const void* Ew, const void* Ep, void* e, int rows, int s,
                               int H, int vocab, hipStream_t st) {
  dim3 grid((rows + 3) / 4), blk(256);
  if (dt == DT_BF16)
    hipLaunchKernelGGL(embed_gather_kernel<bf16>, grid, blk, 0, st, ids, (const bf16*)Ew, (const bf16*)Ep, (bf16*)e,
                       rows, s, H, vocab);
  else
    hipLaunchKernelGGL(embed_gather_kernel<float>, grid, blk, 0, st, ids, (const float*)Ew, (const float*)Ep,
                       (float*)e, rows, s, H, vocab);
  return hipGetLastError();
}

template <typename T>
static hipError_t embed_bwd_t(const int32_t* ids, const T* de, float* dEw, float* dEp, int b, int s, int H, int vocab,
                              int nmb, hipStream_t st) {
  const int rows = b * s, n = (H + 64 * (16 / (int)sizeof(T)) - 1) / (64 * (16 / (int)sizeof(T)));
  dim3 grid((rows * nmb + 3) / 4), blk(256);
#define ESC(N) hipLaunchKernelGGL((embed_scatter_kernel<T, N>), grid, blk, 0, st, ids, de, dEw, rows, nmb, H, vocab)
  if (n <= 1) ESC(1);
  else if (n <= 2) ESC(2);
  else if (n <= 4) ESC(4);
  else return hipErrorInvalidValue;   // wider rows than a stage takes
#undef ESC
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 g2((unsigned)(((long)s * H + 255) / 256));
  hipLaunchKernelGGL(embed_pos_grad_kernel<T>, g2, blk, 0, st, de, dEp, b, s, H, nmb);
  return hipGetLastError();
}

hipError_t launch_embed_bwd(Dtype dt, const int32_t* ids, const void* de, float* dEw, float* dEp, int b, int s, int H,
                            int vocab, int nmb, hipStream_t st) {
  return dt == DT_BF16 ? embed_bwd_t<bf16>(ids, (const bf16*)de, dEw, dEp, b, s, H, vocab, nmb, st)
                       : embed_bwd_t<float>(ids, (const float*)de, dEw, dEp, b, s, H, vocab, nmb, st);
}

hipError_t launch_mlm_compact(const int32_t* targets, int T, int nmb, int cap, int np, int vocab, int32_t* rows_idx,
                              int32_t* tgt, int32_t* info, hipStream_t st) {
  hipLaunchKernelGGL(mlm_compact_kernel, dim3(nmb), dim3(1024), 0, st, targets, T, cap, np, vocab, rows_idx, tgt, info);
  return hipGetLastError();
}

hipError_t launch_gather_rows(Dtype dt, const void* src, const int32_t* idx, void* dst, int n, int H, int nsrc, int nmb,
                              hipStream_t st) {
  const int n16 = H * (dt == DT_BF16 ? 2 : 4) / 16;   // rows are whole 16-byte pieces (hidden is a multiple of 8 / 4)
  hipLaunchKernelGGL(gather_rows_kernel, dim3((n + 3) / 4, nmb), dim3(256), 0, st, (const uint4*)src, idx, (uint4*)dst, n, n16, nsrc);
  return hipGetLastError();
}

hipError_t launch_scatter_rows(Dtype dt, const void* src, const int32_t* idx, void* dst, int n, int H, int ndst, int nmb,
                               hipStream_t st) {
  const int n16 = H * (dt == DT_BF16 ? 2 : 4) / 16;
  hipLaunchKernelGGL(scatter_rows_kernel, dim3((n + 3) / 4, nmb), dim3(256), 0, st, (const uint4*)src, idx, (uint4*)dst, n, n16, ndst);
  return hipGetLastError();
}

template <typename T>
static hipError_t mlm_ce_t(const float* logits, const T* bias, const int32_t* rows_idx, const int32_t* tgt, int n, int V,
                           int VP, float loss_scale, T* dz, float* row_loss, hipStream_t st) {
#define CE(N) hipLaunchKernelGGL((mlm_ce_regs_kernel<T, N>), dim3(n), dim3(1024), 0, st, logits, bias, rows_idx, tgt, V, VP, loss_scale, dz, row_loss)
  if (VP <= 4096) CE(1);
  else if (VP <= 8192) CE(2);
  else if (VP <= 16384) CE(4);
  else if (VP <= 32768) CE(8);
  else hipLaunchKernelGGL(mlm_ce_kernel<T>, dim3(n), dim3(256), 0, st, logits, bias, rows_idx, tgt, V, VP, loss_scale, dz, row_loss);
#undef CE
  return hipGetLastError();
}

hipError_t launch_mlm_ce(Dtype dt, const float* logits, const void* bias, const int32_t* rows_idx, const int32_t* tgt,
                         int n, int V, int VP, float loss_scale, void* dz, float* row_loss, hipStream_t st) {
  return dt == DT_BF16 ? mlm_ce_t<bf16>(logits, (const bf16*)bias, rows_idx, tgt, n, V, VP, loss_scale, (bf16*)dz, row_loss, st)
                       : mlm_ce_t<float>(logits, (const float*)bias, rows_idx, tgt, n, V, VP, loss_scale, (float*)dz, row_loss, st);
}

hipError_t launch_loss_sum(const float* row_loss, int n, int nmb, float scale, float* loss_out, hipStream_t st) {
  hipLaunchKernelGGL(loss_sum_kernel, dim3(nmb), dim3(64), 0, st, row_loss, n, scale, loss_out);
  return hipGetLastError();
}

hipError_t launch_mul(Dtype dt, const void* a, const void* b, void* c, long n, hipStream_t st) {
  dim3 grid((unsigned)((n + 255) / 256)), blk(256);
  if (dt == DT_BF16) hipLaunchKernelGGL(mul_kernel<bf16>, grid, blk, 0, st, (const bf16*)a, (const bf16*)b, (bf16*)c, n);
  else hipLaunchKernelGGL(mul_kernel<float>, grid, blk, 0, st, (const float*)a, (const float*)b, (float*)c, n);
  return hipGetLastError();
}

}  // namespace dapple
