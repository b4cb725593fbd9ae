// Self-attention of one encoder layer, forward and backward, without ever
// writing the s x s probability matrix to HBM.
//
//   forward :  ctx = softmax(q k^T / sqrt(d)) v        + row logsumexp (log2 domain)
//   backward:  P = exp2(t - lse),  dP = dctx v^T,  dS = P o (dP - delta),
//              delta = rowsum(dctx o ctx),
//              dv = P^T dctx,  dq = dS k / sqrt(d),  dk = dS^T q / sqrt(d)
//
// MFMA kernels (bf16, d % 8 == 0, d <= 128, any s): a workgroup of 4 waves; each wave owns
// 32 query rows (forward, dq) or 32 key rows (dk/dv) whose fragments stay in
// registers, and streams 64-row blocks of the other side through LDS.  The
// products are oriented so that the accumulator's lane index is the row the wave
// owns: softmax statistics are then per-lane scalars, and the probabilities leave
// the accumulator already laid out as the next MFMA's operand (the contraction
// index is permuted, and the other operand is fetched from LDS with the same
// permutation through the LDS transpose read).  dq and dk/dv are two sets of
// workgroups that each recompute P: no atomics, every sum in a fixed order, so
// results are reproducible bit for bit.  Both sets go out in ONE launch (grid.z
// picks the role) with at most 256 registers per lane, so that a dq and a dk/dv
// workgroup share a compute unit: each is a chain MFMA -> softmax arithmetic ->
// MFMA with one wave per SIMD, and two of them on a SIMD fill each other's waits
// (b=4, s=512, A=16: 39 us as two launches one after the other, 29 us as one).
// Head widths other than 64 and ragged lengths were on the plain kernels before (2 layers of 1024 with heads of 128,
// 2 x 256 tokens, 4 micro-batches: 242 ms per iteration, 0.67 ms now).
// delta = rowsum(dctx o ctx) must exist before either starts: the stage takes it
// from the epilogue of the product that makes dctx (delta_blocks), a caller
// without that product gets it from a small kernel of its own first.
//
// Plain kernels (any dtype and shape): one thread per output element, for shapes neither
// these MFMA kernels nor those of attention_f32.hip take.
#include "device_common.h"
#include "kernels.h"

namespace dapple {

static constexpr float LOG2E = 1.4426950408889634f;

// ------------------------------------------------------------------ plain kernels
template <typename T>
__global__ void attn_fwd_plain(AttnArgs a, float scale2) {
  long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long total = (long)a.b * a.A * a.s * a.d;
  if (idx >= total) return;
  int dd = idx % a.d;
  int qi = (idx / a.d) % a.s;
  int hh = (idx / ((long)a.d * a.s)) % a.A;
  int bi = idx / ((long)a.d * a.s * a.A);
  const T* q = (const T*)a.q + ((long)bi * a.s + qi) * a.H + hh * a.d;
  const T* kb = (const T*)a.k + (long)bi * a.s * a.H + hh * a.d;
  const T* vb = (const T*)a.v + (long)bi * a.s * a.H + hh * a.d;
  float m = -INFINITY;
  for (int j = 0; j < a.s; ++j) {
    float t = 0.f;
    for (int e = 0; e < a.d; ++e) t = fmaf(to_f32(q[e]), to_f32(kb[(long)j * a.H + e]), t);
    m = fmaxf(m, t * scale2);
  }
  float l = 0.f, o = 0.f;
  for (int j = 0; j < a.s; ++j) {
    float t = 0.f;
    for (int e = 0; e < a.d; ++e) t = fmaf(to_f32(q[e]), to_f32(kb[(long)j * a.H + e]), t);
    float p = exp2f(t * scale2 - m);
    l += p;
    o = fmaf(p, to_f32(vb[(long)j * a.H + dd]), o);
  }
  ((T*)a.ctx)[((long)bi * a.s + qi) * a.H + hh * a.d + dd] = from_f32<T>(o / l);
  if (a.ctx32) a.ctx32[((long)bi * a.s + qi) * a.H + hh * a.d + dd] = o / l;
  if (dd == 0) a.lse[((long)bi * a.A + hh) * a.s + qi] = m + log2f(l);
}

template <typename T>
__global__ void attn_delta_kernel(AttnArgs a) {
  long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long total = (long)a.b * a.s * a.A;
  if (idx >= total) return;
  int hh = idx % a.A;
  long row = idx / a.A;  // bi*s + qi
  const T* o = (const T*)a.ctx + row * a.H + hh * a.d;
  const T* g = (const T*)a.dctx + row * a.H + hh * a.d;
  float t = 0.f;
  if (a.ctx32) {
    const float* o32 = a.ctx32 + row * a.H + hh * a.d;
    for (int e = 0; e < a.d; ++e) t = fmaf(o32[e], to_f32(g[e]), t);
  } else {
    for (int e = 0; e < a.d; ++e) t = fmaf(to_f32(o[e]), to_f32(g[e]), t);
  }
  int bi = row / a.s, qi = row % a.s;
  a.delta[((long)bi * a.A + hh) * a.s + qi] = t;
}

// which = 0: dq, 1: dk, 2: dv; one thread per output element
template <typename T>
__global__ void attn_bwd_plain(AttnArgs a, float scale2, float scale, int which) {
  long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long total = (long)a.b * a.A * a.s * a.d;
  if (idx >= total) return;
  int dd = idx % a.d;
  int ri = (idx / a.d) % a.s;
  int hh = (idx / ((long)a.d * a.s)) % a.A;
  int bi = idx / ((long)a.d * a.s * a.A);
  long hb = (long)bi * a.s * a.H + hh * a.d;
  const T *Q = (const T*)a.q + hb, *K = (const T*)a.k + hb, *V = (const T*)a.v + hb, *G = (const T*)a.dctx + hb;
  const float* lse = a.lse + ((long)bi * a.A + hh) * a.s;
  const float* dl = a.delta + ((long)bi * a.A + hh) * a.s;
  float acc = 0.f;
  for (int o = 0; o < a.s; ++o) {
    int qi = which == 0 ? ri : o, kj = which == 0 ? o : ri;
    float t = 0.f, dp = 0.f;
    for (int e = 0; e < a.d; ++e) {
      t = fmaf(to_f32(Q[(long)qi * a.H + e]), to_f32(K[(long)kj * a.H + e]), t);
      dp = fmaf(to_f32(G[(long)qi * a.H + e]), to_f32(V[(long)kj * a.H + e]), dp);
    }
    float p = exp2f(t * scale2 - lse[qi]);
    float ds = p * (dp - dl[qi]);
    if (which == 0) acc = fmaf(ds, to_f32(K[(long)kj * a.H + dd]), acc);
    else if (which == 1) acc = fmaf(ds, to_f32(Q[(long)qi * a.H + dd]), acc);
    else acc = fmaf(p, to_f32(G[(long)qi * a.H + dd]), acc);
  }
  T* out = (T*)(which == 0 ? a.dq : (which == 1 ? a.dk : a.dv));
  out[hb + (long)ri * a.H + dd] = from_f32<T>(which == 2 ? acc : acc * scale);
}

// ------------------------------------------------------------------ MFMA kernels
// D: width of a head's block in LDS and registers (32, 64 or 128; a head of d <= D columns is padded with zeros).
// RAG: some edge is ragged -- s is no multiple of 64 or d is smaller than D: rows and columns outside are read as
//      zeros, their probabilities are zero, and nothing outside is stored.
// P32: the probabilities and dS enter their products as a sum of three bf16 values, which holds all 24 bits of an fp32
//      one; otherwise they are rounded to bf16 once.  (D = 64 with s % 64 == 0 rounds once; every other shape was served
//      by fp32 arithmetic before it had MFMA kernels and keeps it, the library's exp2f with its denormal results too.
//      Against two bf16 values, 16 bits, and the bare v_exp_f32 it costs 1-5% of an iteration, most where attention is
//      most of it: 4 layers of 768, 3 x 200 tokens, 6 micro-batches 2.00 -> 2.01 ms; 2 layers of 1024 with heads of 128,
//      2 x 256 tokens, 4 micro-batches 0.704 -> 0.714; 3 layers of 320, 444 tokens, 4 micro-batches 0.628 -> 0.661.)

// A 64 x D bf16 block sits in LDS as 64 rows of D/8 16-byte chunks, the chunks of row r XOR-swizzled by aswz(r).
// The same block is read two ways -- 128-bit reads along a row (16 lanes = 16 rows at a time) and transpose reads
// down the rows (32 lanes = 4 rows x 64 bytes at a time) -- and LDS has 64 four-byte banks, so either group must
// cover 256 distinct bytes modulo 256.
//   D = 64:  rows of equal parity need distinct chunks (a bijection of (r>>1)&7), and rows r and r+2 must land in
//            different 64-byte halves (bit 2 of the swizzle = bit 1 of r): (r>>1)&7 rotated right by one gives both.
//   D = 128: 16 rows need 16 distinct chunks and 4 neighbouring rows four distinct 64-byte quarters: the two halves
//            of r & 15 swapped.
//   D = 32:  four rows fill 256 bytes; rows r, r+4, r+8, r+12 need distinct chunks: (r>>2)&3.
template <int D>
__device__ __forceinline__ int aswz(int r) {
  if (D == 64) {
    int x = (r >> 1) & 7;
    return ((x & 1) << 2) | (x >> 1);
  }
  if (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  return (r >> 2) & 3;
}

// The streamed side: blocks of 64 rows of two matrices X and Y (keys and values; queries and output gradients) go
// through a ring of NS blocks in LDS, requested NS - 1 blocks ahead with loads that write LDS directly.  (Through
// registers, one block ahead, every block waited for memory: a block's arithmetic is about 0.6 us, a request takes
// longer.)  1 KiB per wave instruction in lane order, so the swizzle is applied to WHICH chunk a lane fetches; rows
// past the end lie beyond the buffer's record count and read as zero, columns past d get an offset out of range.
// A wave owns PER consecutive instructions of one of the two matrices.
typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int D, int NW, int NS_, bool STATS>
struct Ring {
  static constexpr int NS = NS_, IPM = D / 8, PER = 2 * IPM / NW;          // instructions per matrix and block; per wave
  static constexpr int Y_OFF = 64 * D * 2, S_OFF = 2 * Y_OFF;              // X, Y, then rows of 64 fp32 (STATS)
  static constexpr int SROWS = NW > 4 ? NW : 4, STAGE = S_OFF + (STATS ? SROWS * 256 : 0), BYTES = NS * STAGE;
  static constexpr int SPW = STATS ? SROWS / NW : 0;   // rows of the statistics per wave
  static constexpr int BIAS = 3072, LOADS = PER + SPW;
  static_assert(PER <= IPM && (PER == 2 || PER % 4 == 0), "a wave's share lies in one matrix");
  static_assert((NS - 2) * LOADS < 64, "vmcnt is a 6-bit counter");
  int voff[PER];
  i32x4 rs, st[SPW ? SPW : 1];   // buffer resources: the wave's matrix; its rows of the statistics
  int step, left, left0, sleft[SPW ? SPW : 1], m0w, m0s;
  uint64_t base0, stat0[SPW ? SPW : 1];
  // g: the wave's matrix (head's first column of row 0); ld in elements; stat(r): row r of the statistics, fp32 per row
  // of X and Y, or NULL (reads zero)
  template <typename F>
  __device__ __forceinline__ void init(const bf16* g, int ld, int s, int d, int wave, int lane, F&& stat) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int pos = ((wave * PER + j) % IPM) * 64 + lane, r = pos / (D / 8), c = (pos % (D / 8)) ^ aswz<D>(r);
      voff[j] = c * 8 < d ? (r * ld + c * 8) * 2 + BIAS - (j % 4) * 1024 : (int)0x80000000;
    }
    set(rs, (uint64_t)g - BIAS);
    step = 64 * ld * 2;
    left = left0 = ((s - 1) * ld + d) * 2;
    base0 = (uint64_t)g - BIAS;
    m0w = __builtin_amdgcn_readfirstlane(wave * PER * 1024);
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      const float* p = stat(wave + NW * i);
      stat0[i] = (uint64_t)p;
      set(st[i], (uint64_t)p);
      sleft[i] = p ? s * 4 : 0;
    }
    m0s = __builtin_amdgcn_readfirstlane(S_OFF + wave * 256);
  }
  static __device__ __forceinline__ void set(i32x4& r, uint64_t p) {
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    r[3] = 0x00020000;   // raw buffer, 32-bit data format
  }
  // request the next block into stage `stage`.  Inline assembly, and the waits counted by hand, for the reasons given
  // at OperandTile::load_group in gemm_mfma.h (which also has the wait states).
  __device__ __forceinline__ void request(int stage, int lane) {
    const int base = __builtin_amdgcn_readfirstlane(stage * STAGE);
    rs[2] = __builtin_amdgcn_readfirstlane(left > 0 ? left + BIAS : 0);
    const int mw = __builtin_amdgcn_readfirstlane(base + m0w);
    if constexpr (PER == 2) {
      asm volatile(
          "s_nop 4\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\t"
          "buffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
          "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds"
          :
          : "s"(mw), "v"(voff[0]), "v"(voff[1]), "s"(rs)
          : "memory", "m0");
    } else {
#pragma unroll
      for (int j = 0; j < PER; j += 4)
        asm volatile(
            "s_nop 4\n\ts_add_u32 m0, %0, %1\n\ts_nop 0\n\t"
            "buffer_load_dwordx4 %2, %6, 0 offen lds\n\t"
            "buffer_load_dwordx4 %3, %6, 0 offen offset:1024 lds\n\t"
            "buffer_load_dwordx4 %4, %6, 0 offen offset:2048 lds\n\t"
            "buffer_load_dwordx4 %5, %6, 0 offen offset:3072 lds"
            :
            : "s"(mw), "s"(j * 1024), "v"(voff[j]), "v"(voff[j + 1]), "v"(voff[j + 2]), "v"(voff[j + 3]), "s"(rs)
            : "memory", "m0", "scc");
    }
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      st[i][2] = __builtin_amdgcn_readfirstlane(sleft[i] > 0 ? sleft[i] : 0);
      const int ms = __builtin_amdgcn_readfirstlane(base + m0s + i * NW * 256);
      const int off = lane * 4;
      asm volatile(
          "s_nop 4\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\t"
          "buffer_load_dword %1, %2, 0 offen lds"
          :
          : "s"(ms), "v"(off), "s"(st[i])
          : "memory", "m0");
      set(st[i], (((uint64_t)(uint32_t)st[i][1] << 32) | (uint32_t)st[i][0]) + 256);
      sleft[i] -= 256;
    }
    set(rs, (((uint64_t)(uint32_t)rs[1] << 32) | (uint32_t)rs[0]) + (uint64_t)step);
    left -= step;
  }
  // the next block requested is the first one again
  __device__ __forceinline__ void rewind(int s) {
    set(rs, base0);
    left = left0;
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      set(st[i], stat0[i]);
      sleft[i] = stat0[i] ? s * 4 : 0;
    }
  }
  // what is requested from here on reads nothing
  __device__ __forceinline__ void stop() {
    left = 0;
#pragma unroll
    for (int i = 0; i < SPW; ++i) sleft[i] = 0;
  }
  // every wave's part of the oldest block is in LDS, and every wave is done with the block before it.  MORE: requests of
  // this wave's besides the ring's, issued since the one that is waited for
  template <int MORE = 0>
  static __device__ __forceinline__ void wait() {
    constexpr int N = (NS - 2) * LOADS + MORE;
    static_assert(N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);   // vmcnt(N), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
};
// operand fragment, contraction index contiguous in LDS: rows r0 + (lane&31), k = 16 kk + 8 (lane>>5) + e
template <int D>
__device__ __forceinline__ bf16x8 frag_rows(const bf16* S, int r0, int kk, int lane) {
  int r = r0 + (lane & 31), kc = kk * 2 + (lane >> 5);
  return *(const bf16x8*)(S + r * D + ((kc ^ aswz<D>(r)) << 3));
}
// operand fragment, contraction index along LDS rows: column c0 + (lane&31); element e < 4 is
// LDS row k0 + 4 (lane>>5) + e, element 4 + e is LDS row k0 + 8 + 4 (lane>>5) + e -- the order
// in which a 32x32 accumulator hands its rows to a lane
template <int D>
__device__ __forceinline__ bf16x8 frag_cols(const bf16* S, int c0, int k0, int lane) {
  int i16 = lane & 15, g16 = (lane >> 4) & 1, h = lane >> 5;
  int r = k0 + 4 * h + (i16 >> 2);
  int col = c0 + 16 * g16 + 4 * (i16 & 3);
  const bf16* p0 = S + r * D + (((col >> 3) ^ aswz<D>(r)) << 3) + (col & 7);
  const bf16* p1 = S + (r + 8) * D + (((col >> 3) ^ aswz<D>(r + 8)) << 3) + (col & 7);
  return join8(lds_read_tr16(p0), lds_read_tr16(p1));
}
// global fragment of a row the wave owns: row r (or zeros), k = 16 kk + 8 (lane>>5) + e
template <bool RAG>
__device__ __forceinline__ bf16x8 frag_global(const bf16* base, long row, bool ok, int ld, int kk, int lane, int d) {
  const int k = kk * 16 + 8 * (lane >> 5);
  if (!ok || (RAG && k >= d)) {
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (bf16)0.f;
    return z;
  }
  return *(const bf16x8*)(base + row * ld + k);
}
// accumulator rows 16 ks .. 16 ks + 15 of a 32-row block, as the k-permuted operand
__device__ __forceinline__ bf16x8 acc_to_operand(const float (&p)[16], int ks) {
  bf16x8 f;
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = (bf16)p[8 * ks + e];
  return f;
}
// two fp32 values as bf16 in one register, and what rounding left of them (the differences are exact)
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
__device__ __forceinline__ unsigned take_bf16(float& a, float& b) {
  const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
  a -= __builtin_bit_cast(float, u << 16);
  b -= __builtin_bit_cast(float, u & 0xffff0000u);
  return u;
}
// accumulator rows 16 ks .. 16 ks + 15 as a sum of three such operands.  (Pair by pair in whole registers: element by
// element the compiler converts every value once to pack it and once more to subtract it: the last of the stages above 0.673 ms.)
__device__ __forceinline__ void acc_to_operands(const float (&p)[16], int ks, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
  typedef unsigned u32x4 __attribute__((__vector_size__(4 * sizeof(unsigned))));
  u32x4 h, m, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = p[8 * ks + 2 * e], b = p[8 * ks + 2 * e + 1];
    h[e] = take_bf16(a, b);
    m[e] = take_bf16(a, b);
    l[e] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
  }
  hi = __builtin_bit_cast(bf16x8, h);
  mid = __builtin_bit_cast(bf16x8, m);
  lo = __builtin_bit_cast(bf16x8, l);
}

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)

// delta of query row qi of sequence bi, head hh: from [b, A, s], or the head's d/32 blocks of 32 columns
// out of [H/32][b*s]
template <int D>
__device__ __forceinline__ float delta_at(const AttnArgs& a, int bi, int hh, int qi) {
  if (a.delta_blocks) {   // only where d == D
    const long T = (long)a.b * a.s, row = (long)bi * a.s + qi;
    float t = a.delta_blocks[(D / 32 * hh) * T + row];
#pragma unroll
    for (int j = 1; j < D / 32; ++j) t += a.delta_blocks[(D / 32 * hh + j) * T + row];
    return t;
  }
  return a.delta[((long)bi * a.A + hh) * a.s + qi];
}

// 2^x of every element.  Where a probability is rounded to bf16 anyway (P32 unset) the bare v_exp_f32: one below 2^-126
// may as well be zero there.  Otherwise the library's exp2f, which wraps it in four more instructions that scale denormal
// results -- and gives its bits where there are none, so they are spent only where an element of the wave needs them
// (2 layers of 768, heads of 32, 4 x 256 tokens, 4 micro-batches: 0.865 ms with exp2f always, 0.841 so).
// CHECK unset: spent always, where the check's registers would spill (dk and dv of 64-wide heads in workgroups of two
// waves; more registers per wave there are slower still).
template <bool P32, bool CHECK, int N>
__device__ __forceinline__ void exp2_all(float (&x)[N]) {
  if constexpr (P32 && !CHECK) {
#pragma unroll
    for (int v = 0; v < N; ++v) x[v] = exp2f(x[v]);
    return;
  }
  if constexpr (P32) {
    float least = x[0];
#pragma unroll
    for (int v = 1; v < N; ++v) least = fminf(least, x[v]);
    if (__builtin_amdgcn_ballot_w64(least < -126.f)) {
#pragma unroll
      for (int v = 0; v < N; ++v) x[v] = exp2f(x[v]);
      return;
    }
  }
#pragma unroll
  for (int v = 0; v < N; ++v) x[v] = __builtin_amdgcn_exp2f(x[v]);
}
template <bool P32>
__device__ __forceinline__ float exp2_of(float x) {
  return P32 ? exp2f(x) : __builtin_amdgcn_exp2f(x);
}

// max / sum of the two half waves' values (a row's 64 keys sit in lanes l and l + 32), in both; v_permlane32_swap is an
// ordinary vector instruction where a shuffle is a trip through the LDS crossbar
__device__ __forceinline__ float halves_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}

// A wave's 32 rows x 32 NDB columns of an output (t: rows = columns of the head, column = the lane's row) times f, through a
// piece of LDS of the wave's own into whole rows: straight from the accumulators a store is 16 bytes (32 of an fp32 copy)
// of each of 32 rows, and the L2 takes every line in eight pieces.  rows: valid rows; d: columns of the head.
// C32 (may be NULL): an fp32 copy; FAR: it is not read again soon enough to be kept in a cache (see store_c in gemm_mfma.h).
template <int NDB, bool FAR = false>
struct OutTile {
  static constexpr int W = 32 * NDB, LD = W + 4, BYTES = 32 * LD * 4;
  static constexpr int RS = 64 / (W / 4);   // rows per instruction
  // Vector stores of C by a wave whose 32 rows and W columns are all valid, C32 aside.  A caller's wait may count on as many
  // behind an older request: one instruction per RS rows, and no way past it.
  static constexpr int STORES = 32 / RS;
  static __device__ __forceinline__ void store(float* S, const f32x16* t, float f, bf16* C, float* C32, long ld, int rows, int d, int lane) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int blk = 0; blk < 4; ++blk)
        *(f32x4*)(S + (lane & 31) * LD + db * 32 + 8 * blk + 4 * (lane >> 5)) =
            f32x4{t[db][4 * blk], t[db][4 * blk + 1], t[db][4 * blk + 2], t[db][4 * blk + 3]} * f;
    __builtin_amdgcn_wave_barrier();   // (private to the wave, whose LDS accesses execute in order)
    const int r = lane / (W / 4), c = lane % (W / 4) * 4;
#pragma unroll
    for (int u = 0; u < STORES; ++u) {
      const int i = u * RS;
      const f32x4 v = *(const f32x4*)(S + (i + r) * LD + c);
      if (i + r < rows && c < d) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16)v[e];
        *(bf16x4*)(C + (i + r) * ld + c) = o;
        if (C32) {
          if (FAR) __builtin_nontemporal_store(v, (f32x4*)(C32 + (i + r) * ld + c));
          else *(f32x4*)(C32 + (i + r) * ld + c) = v;
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
};

// NW: waves per workgroup (4, or 2 where the grid is small), each with 32 query rows
template <int D, bool RAG, bool P32, int NW>
__global__ __launch_bounds__(64 * NW, D == 128 ? 1 : 2) void attn_fwd_mfma(AttnArgs a, float scale2) {
  constexpr int NKK = D / 16, NDB = D / 32;
  typedef Ring<D, NW, D == 128 ? 2 : 3, false> R;
  extern __shared__ __attribute__((aligned(1024))) unsigned char asm_[];
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bi = (a.head0 + blockIdx.y) / a.A, hh = (a.head0 + blockIdx.y) % a.A;
  const int d = RAG ? a.d : D;
  const long hb = (long)bi * a.s * a.H + hh * d;
  const bf16 *Q = (const bf16*)a.q + hb, *K = (const bf16*)a.k + hb, *V = (const bf16*)a.v + hb;
  const int qrow = blockIdx.x * (32 * NW) + wave * 32 + (lane & 31);
  const bool qok = qrow < a.s;
  const int nkb = RAG ? (a.s + 63) / 64 : a.s / 64;
  bf16x8 qf[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) qf[kk] = frag_global<RAG>(Q, qrow, qok, a.H, kk, lane, d);
  R ring;
  ring.init(wave < NW / 2 ? K : V, a.H, a.s, d, wave, lane, [](int) { return (const float*)nullptr; });
  __builtin_amdgcn_s_waitcnt(0x0F70);   // the query fragments are here: the counts below are the ring's alone
#pragma unroll
  for (int t = 0; t < R::NS - 1; ++t) ring.request(t, lane);

  float m = -INFINITY, l = 0.f;
  f32x16 o[NDB];  // rows d = 32 dblk + 8 blk + 4 h + e, column = the lane's query
#pragma unroll
  for (int db = 0; db < NDB; ++db) o[db] = zero16();

  int stage = 0;
  for (int kb = 0; kb < nkb; ++kb) {
    R::wait();
    ring.request(stage == 0 ? R::NS - 1 : stage - 1, lane);   // (past the last block: reads nothing)
    const bf16 *Ks = (const bf16*)(asm_ + stage * R::STAGE), *Vs = (const bf16*)((const unsigned char*)Ks + R::Y_OFF);
    stage = stage + 1 == R::NS ? 0 : stage + 1;
    float p[2][16];
    float mx = -INFINITY;
    // All LDS reads of a phase are issued before its first MFMA (left to itself the compiler
    // reuses one register set and waits for every read in turn): the key fragments, then the
    // value fragments, which land while the softmax arithmetic runs.  (D = 128: by halves, for registers.)
    bf16x8 kf[2][NKK], vf[4][NDB];
    constexpr bool ALL = D <= 64;
    if (ALL) {
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) kf[kb2][kk] = frag_rows<D>(Ks, kb2 * 32, kk, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
      if (!ALL) {
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) kf[kb2][kk] = frag_rows<D>(Ks, kb2 * 32, kk, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
      f32x16 sa = zero16();  // rows: key 32 kb2 + 8 blk + 4 h + e, column: query
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) sa = MFMA(kf[kb2][kk], qf[kk], sa);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        p[kb2][v] = sa[v];
        mx = fmaxf(mx, sa[v]);
      }
    }
    if (RAG && kb + 1 == nkb) {   // without the keys beyond the last
      mx = -INFINITY;
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          if (kb * 64 + kb2 * 32 + 8 * (v >> 2) + 4 * h + (v & 3) >= a.s) p[kb2][v] = -INFINITY;
          mx = fmaxf(mx, p[kb2][v]);
        }
    }
    if (ALL) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int db = 0; db < NDB; ++db) vf[ks][db] = frag_cols<D>(Vs, db * 32, ks * 16, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the maximum is taken over the raw products (the scale is positive): one multiply-add per logit, not two steps
    const float mn = fmaxf(m, halves_max(mx) * scale2);
    const float alpha = exp2_of<P32>(m - mn);
    float rs = 0.f;
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
      if (P32) {
#pragma unroll
        for (int v = 0; v < 16; ++v) p[kb2][v] = fmaf(p[kb2][v], scale2, -mn);
        exp2_all<true, true>(p[kb2]);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if (!P32) p[kb2][v] = __builtin_amdgcn_exp2f(fmaf(p[kb2][v], scale2, -mn));
        rs += p[kb2][v];
      }
    }
    l = l * alpha + halves_sum(rs);
    m = mn;
    // the running maximum of most rows settles after the first key blocks: skip the rescale of
    // the accumulator registers when no lane of the wave needs it (alpha == 1 exactly)
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      bf16x8 pf, pm, pl;
      if (P32) acc_to_operands(p[ks >> 1], ks & 1, pf, pm, pl);
      else pf = acc_to_operand(p[ks >> 1], ks & 1);
      if (!ALL) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) vf[ks][db] = frag_cols<D>(Vs, db * 32, ks * 16, lane);
      }
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[db] = MFMA(vf[ks][db], pf, o[db]);
      if (P32) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db] = MFMA(vf[ks][db], pm, o[db]);
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db] = MFMA(vf[ks][db], pl, o[db]);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // the ring's last requests (they read nothing) before the wave may end
  const float inv = 1.0f / l;
  if constexpr (D <= 64) {
    typedef OutTile<NDB, NW == 4> Out;
    static_assert(NW * Out::BYTES <= R::BYTES, "the output's staging lies where the ring was");
    __syncthreads();   // every wave is done with the ring, and its requests
    const int row0 = blockIdx.x * (32 * NW) + wave * 32;
    const long o0 = hb + (long)row0 * a.H;
    Out::store((float*)(asm_ + wave * Out::BYTES), o, inv, (bf16*)a.ctx + o0, a.ctx32 ? a.ctx32 + o0 : nullptr, a.H, a.s - row0, d, lane);
  } else if (qok) {
    bf16* C = (bf16*)a.ctx + hb + (long)qrow * a.H;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        const int col = db * 32 + 8 * blk + 4 * h;
        if (RAG && col >= d) continue;
        bf16x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (bf16)(o[db][4 * blk + e] * inv);
        *(bf16x4*)(C + col) = ov;
        if (a.ctx32)
          *(float4*)(a.ctx32 + hb + (long)qrow * a.H + col) =
              make_float4(o[db][4 * blk] * inv, o[db][4 * blk + 1] * inv, o[db][4 * blk + 2] * inv, o[db][4 * blk + 3] * inv);
      }
  }
  if (qok && h == 0) a.lse[((long)bi * a.A + hh) * a.s + qrow] = m + log2f(l);
}

// dk, dv: the wave owns 32 key rows; query blocks of 64 stream through LDS with their lse and delta (the two blocks
// of 32 columns a head of 64 has are added where they are read)
template <int D, bool RAG, bool P32, int NW, typename R>
__device__ __forceinline__ void attn_dkdv_body(const AttnArgs& a, float scale2, float scale, unsigned char* sm) {
  constexpr int NKK = D / 16, NDB = D / 32;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bi = (a.head0 + blockIdx.y) / a.A, hh = (a.head0 + blockIdx.y) % a.A;
  const int d = RAG ? a.d : D;
  const long hb = (long)bi * a.s * a.H + hh * d;
  const bf16 *Q = (const bf16*)a.q + hb, *K = (const bf16*)a.k + hb, *V = (const bf16*)a.v + hb,
             *G = (const bf16*)a.dctx + hb;
  const float* lse = a.lse + ((long)bi * a.A + hh) * a.s;
  const int krow = blockIdx.x * (32 * NW) + wave * 32 + (lane & 31);
  const bool kok = krow < a.s;

  bf16x8 kf[NKK], vf[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    kf[kk] = frag_global<RAG>(K, krow, kok, a.H, kk, lane, d);
    vf[kk] = frag_global<RAG>(V, krow, kok, a.H, kk, lane, d);
  }
  f32x16 dv[NDB], dk[NDB];  // rows d, column = the lane's key
#pragma unroll
  for (int db = 0; db < NDB; ++db) dv[db] = dk[db] = zero16();
  const int nqb = RAG ? (a.s + 63) / 64 : a.s / 64;
  // row 0 of the statistics: lse; 1 and 2: delta, or its blocks of 32 columns; 3: unused.
  // A query beyond the last has zero rows, lse 0 and delta 0: probability 1 times a zero row, dS = 0.
  const long T = (long)a.b * a.s;
  const float *d0 = a.delta + ((long)bi * a.A + hh) * a.s, *d1 = nullptr;
  if (a.delta_blocks) {
    d0 = a.delta_blocks + (long)(D / 32 * hh) * T + (long)bi * a.s;
    if (D >= 64) d1 = d0 + T;
  }
  R ring;
  ring.init(wave < NW / 2 ? Q : G, a.H, a.s, d, wave, lane, [&](int r) { return r == 0 ? lse : (r == 1 ? d0 : (r == 2 ? d1 : nullptr)); });
  __builtin_amdgcn_s_waitcnt(0x0F70);   // the key and value fragments are here: the counts below are the ring's alone
#pragma unroll
  for (int t = 0; t < R::NS - 1; ++t) ring.request(t, lane);

  int stage = 0;
  for (int qb = 0; qb < nqb; ++qb) {
    R::wait();
    ring.request(stage == 0 ? R::NS - 1 : stage - 1, lane);
    const bf16 *Qs = (const bf16*)(sm + stage * R::STAGE), *Gs = (const bf16*)((const unsigned char*)Qs + R::Y_OFF);
    const float *Ls = (const float*)((const unsigned char*)Qs + R::S_OFF), *Ds = Ls + 64;
    stage = stage + 1 == R::NS ? 0 : stage + 1;
#pragma unroll
    for (int qb2 = 0; qb2 < 2; ++qb2) {
      // every LDS read of a phase before its first MFMA (see attn_fwd_mfma)
      bf16x8 qf[NKK], gf[NKK], gc[2][NDB], qc[2][NDB];
      float4 L4s[4], D4s[4];
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        qf[kk] = frag_rows<D>(Qs, qb2 * 32, kk, lane);
        gf[kk] = frag_rows<D>(Gs, qb2 * 32, kk, lane);
      }
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        L4s[blk] = *(const float4*)(Ls + qb2 * 32 + 8 * blk + 4 * h);
        D4s[blk] = *(const float4*)(Ds + qb2 * 32 + 8 * blk + 4 * h);
        if (D >= 64) {   // the second block of delta (zero where delta comes whole)
          const float4 x = *(const float4*)(Ds + 64 + qb2 * 32 + 8 * blk + 4 * h);
          D4s[blk].x += x.x; D4s[blk].y += x.y; D4s[blk].z += x.z; D4s[blk].w += x.w;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      f32x16 sa = zero16(), dp = zero16();  // rows: query 32 qb2 + 8 blk + 4 h + e, column: key
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        sa = MFMA(qf[kk], kf[kk], sa);
        dp = MFMA(gf[kk], vf[kk], dp);
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          gc[ks][db] = frag_cols<D>(Gs, db * 32, qb2 * 32 + ks * 16, lane);
          qc[ks][db] = frag_cols<D>(Qs, db * 32, qb2 * 32 + ks * 16, lane);
        }
      __builtin_amdgcn_sched_barrier(0);
      float p[16], ds[16];   // (dP - delta first: its registers are free again before the exponentials)
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        const float Lv[4] = {L4s[blk].x, L4s[blk].y, L4s[blk].z, L4s[blk].w}, Dv[4] = {D4s[blk].x, D4s[blk].y, D4s[blk].z, D4s[blk].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[4 * blk + e] = fmaf(sa[4 * blk + e], scale2, -Lv[e]);
          ds[4 * blk + e] = dp[4 * blk + e] - Dv[e];
        }
      }
      exp2_all<P32, D != 64 || NW == 4>(p);
#pragma unroll
      for (int v = 0; v < 16; ++v) ds[v] *= p[v];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf16x8 pf, pm, pl, dsf, dsm, dsl;
        if (P32) {
          acc_to_operands(p, ks, pf, pm, pl);
          acc_to_operands(ds, ks, dsf, dsm, dsl);
        } else {
          pf = acc_to_operand(p, ks);
          dsf = acc_to_operand(ds, ks);
        }
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          dv[db] = MFMA(gc[ks][db], pf, dv[db]);
          dk[db] = MFMA(qc[ks][db], dsf, dk[db]);
        }
        if (P32) {
#pragma unroll
          for (int db = 0; db < NDB; ++db) {
            dv[db] = MFMA(gc[ks][db], pm, dv[db]);
            dk[db] = MFMA(qc[ks][db], dsm, dk[db]);
          }
#pragma unroll
          for (int db = 0; db < NDB; ++db) {
            dv[db] = MFMA(gc[ks][db], pl, dv[db]);
            dk[db] = MFMA(qc[ks][db], dsl, dk[db]);
          }
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  if constexpr (D <= 64) {   // (as in attn_fwd_mfma)
    typedef OutTile<NDB> Out;
    static_assert(NW * Out::BYTES <= R::BYTES, "the output's staging lies where the ring was");
    __syncthreads();
    const int row0 = blockIdx.x * (32 * NW) + wave * 32;
    const long o0 = hb + (long)row0 * a.H;
    float* const S = (float*)(sm + wave * Out::BYTES);
    Out::store(S, dk, scale, (bf16*)a.dk + o0, nullptr, a.H, a.s - row0, d, lane);
    Out::store(S, dv, 1.f, (bf16*)a.dv + o0, nullptr, a.H, a.s - row0, d, lane);
  } else if (kok) {
    bf16* DK = (bf16*)a.dk + hb + (long)krow * a.H;
    bf16* DV = (bf16*)a.dv + hb + (long)krow * a.H;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        const int col = db * 32 + 8 * blk + 4 * h;
        if (RAG && col >= d) continue;
        bf16x4 o1, o2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o1[e] = (bf16)(dk[db][4 * blk + e] * scale);
          o2[e] = (bf16)dv[db][4 * blk + e];
        }
        *(bf16x4*)(DK + col) = o1;
        *(bf16x4*)(DV + col) = o2;
      }
  }
}

// dq: the wave owns 32 query rows; key blocks of 64 stream through LDS
template <int D, bool RAG, bool P32, int NW, typename R>
__device__ __forceinline__ void attn_dq_body(const AttnArgs& a, float scale2, float scale, unsigned char* sm) {
  constexpr int NKK = D / 16, NDB = D / 32;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bi = (a.head0 + blockIdx.y) / a.A, hh = (a.head0 + blockIdx.y) % a.A;
  const int d = RAG ? a.d : D;
  const long hb = (long)bi * a.s * a.H + hh * d;
  const bf16 *Q = (const bf16*)a.q + hb, *K = (const bf16*)a.k + hb, *V = (const bf16*)a.v + hb,
             *G = (const bf16*)a.dctx + hb;
  const int qrow = blockIdx.x * (32 * NW) + wave * 32 + (lane & 31);
  const bool qok = qrow < a.s;
  const float Lq = qok ? a.lse[((long)bi * a.A + hh) * a.s + qrow] : 0.f;

  const float Dq = qok ? delta_at<D>(a, bi, hh, qrow) : 0.f;
  bf16x8 qf[NKK], gf[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    qf[kk] = frag_global<RAG>(Q, qrow, qok, a.H, kk, lane, d);
    gf[kk] = frag_global<RAG>(G, qrow, qok, a.H, kk, lane, d);
  }
  f32x16 dq[NDB];  // rows d, column = the lane's query
#pragma unroll
  for (int db = 0; db < NDB; ++db) dq[db] = zero16();
  const int nkb = RAG ? (a.s + 63) / 64 : a.s / 64;
  R ring;
  ring.init(wave < NW / 2 ? K : V, a.H, a.s, d, wave, lane, [](int) { return (const float*)nullptr; });   // (the statistics' loads read nothing)
  __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
  for (int t = 0; t < R::NS - 1; ++t) ring.request(t, lane);

  int stage = 0;
  for (int kb = 0; kb < nkb; ++kb) {
    R::wait();
    ring.request(stage == 0 ? R::NS - 1 : stage - 1, lane);
    const bf16 *Ks = (const bf16*)(sm + stage * R::STAGE), *Vs = (const bf16*)((const unsigned char*)Ks + R::Y_OFF);
    stage = stage + 1 == R::NS ? 0 : stage + 1;
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
      // every LDS read of a phase before its first MFMA (see attn_fwd_mfma)
      bf16x8 kr[NKK], vr[NKK], kc[2][NDB];
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        kr[kk] = frag_rows<D>(Ks, kb2 * 32, kk, lane);
        vr[kk] = frag_rows<D>(Vs, kb2 * 32, kk, lane);
      }
      __builtin_amdgcn_sched_barrier(0);
      f32x16 sa = zero16(), dp = zero16();  // rows: key 32 kb2 + 8 blk + 4 h + e, column: query
#pragma unroll
      for (int kk = 0; kk < NKK; ++kk) {
        sa = MFMA(kr[kk], qf[kk], sa);
        dp = MFMA(vr[kk], gf[kk], dp);
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int db = 0; db < NDB; ++db) kc[ks][db] = frag_cols<D>(Ks, db * 32, kb2 * 32 + ks * 16, lane);
      __builtin_amdgcn_sched_barrier(0);
      float ds[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) ds[v] = fmaf(sa[v], scale2, -Lq);
      exp2_all<P32, true>(ds);
#pragma unroll
      for (int v = 0; v < 16; ++v) ds[v] *= dp[v] - Dq;
      // a key beyond the last: its logit 0 may lie far above the row's logsumexp, so it is masked, not multiplied away
      if (RAG && kb + 1 == nkb) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kb * 64 + kb2 * 32 + 8 * (v >> 2) + 4 * h + (v & 3) >= a.s) ds[v] = 0.f;
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf16x8 dsf, dsm, dsl;
        if (P32) acc_to_operands(ds, ks, dsf, dsm, dsl);
        else dsf = acc_to_operand(ds, ks);
#pragma unroll
        for (int db = 0; db < NDB; ++db) dq[db] = MFMA(kc[ks][db], dsf, dq[db]);
        if (P32) {
#pragma unroll
          for (int db = 0; db < NDB; ++db) dq[db] = MFMA(kc[ks][db], dsm, dq[db]);
#pragma unroll
          for (int db = 0; db < NDB; ++db) dq[db] = MFMA(kc[ks][db], dsl, dq[db]);
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  if constexpr (D <= 64) {   // (as in attn_fwd_mfma)
    typedef OutTile<NDB> Out;
    __syncthreads();
    const int row0 = blockIdx.x * (32 * NW) + wave * 32;
    Out::store((float*)(sm + wave * Out::BYTES), dq, scale, (bf16*)a.dq + hb + (long)row0 * a.H, nullptr, a.H, a.s - row0, d, lane);
  } else if (qok) {
    bf16* DQ = (bf16*)a.dq + hb + (long)qrow * a.H;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        const int col = db * 32 + 8 * blk + 4 * h;
        if (RAG && col >= d) continue;
        bf16x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (bf16)(dq[db][4 * blk + e] * scale);
        *(bf16x4*)(DQ + col) = ov;
      }
  }
}

// delta [b, A, s] for the MFMA backward of a caller that has no product in front to leave it: one wave per row
// of dctx / ctx, a lane takes 8 consecutive columns, a head (d = 32, 64 or 128 columns) is d/8 consecutive lanes
template <int D>
__global__ __launch_bounds__(256) void attn_delta_rows(AttnArgs a) {
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= (long)a.b * a.s) return;
  const int bi = (int)(row / a.s), qi = (int)(row % a.s);
  for (int c0 = 0; c0 < a.H; c0 += 512) {
    const int col = c0 + lane * 8;
    float t = 0.f;
    if (col < a.H) {
      const bf16x8 g = *(const bf16x8*)((const bf16*)a.dctx + row * a.H + col);
      if (a.ctx32) {
        const float4 lo = *(const float4*)(a.ctx32 + row * a.H + col), hi = *(const float4*)(a.ctx32 + row * a.H + col + 4);
        const float ov[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) t = fmaf((float)g[e], ov[e], t);
      } else {
        const bf16x8 o = *(const bf16x8*)((const bf16*)a.ctx + row * a.H + col);
#pragma unroll
        for (int e = 0; e < 8; ++e) t = fmaf((float)g[e], (float)o[e], t);
      }
    }
#pragma unroll
    for (int x = 1; x < D / 8; x <<= 1) t += __shfl_xor(t, x, 64);
    if (col < a.H && lane % (D / 8) == 0) a.delta[((long)bi * a.A + col / D) * a.s + qi] = t;
  }
}

// both roles in one launch: grid.z = 0 the dq workgroups, 1 the dk/dv workgroups.  At most 256 registers per lane up
// to D = 64, so that a workgroup of each role shares a compute unit; D = 128 keeps twice the accumulators.
template <int D, int NW>
struct BwdRing {
  typedef Ring<D, NW, D == 128 ? 2 : 3, true> R;
};
template <int D, bool RAG, bool P32, int NW>
__global__ __launch_bounds__(64 * NW, D <= 64 ? 2 : 1) void attn_bwd_mfma(AttnArgs a, float scale2, float scale) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char asm_[];
  typedef typename BwdRing<D, NW>::R R;
  if (blockIdx.z == 0) attn_dq_body<D, RAG, P32, NW, R>(a, scale2, scale, asm_);
  else attn_dkdv_body<D, RAG, P32, NW, R>(a, scale2, scale, asm_);
}

// The backward with S and dP computed once (heads of 64, whole blocks of 64, 256 to 512 rows).  One workgroup of eight
// waves per head.  Waves 0-3 own 32 keys each, 128 in all, keep their dK and dV in registers while the queries stream
// past in blocks of 64, and leave dS in LDS; waves 4-7, a block behind, own 32 queries x 32 columns of every block and
// add dS K to their part of dQ, which they hold for the whole sequence (128 registers).  Then the next 128 keys.
// The two kinds of workgroups of attn_bwd_mfma do seven products where these do five, and every exponential twice: 16 x
// 512 rows, 16 heads 87 -> 70 us in the trace of an iteration.  Bound by the first kind's chain of products, exponentials and products
// with one wave of each kind per SIMD (matrix pipes 25%, vector units 25%, LDS 30% busy); dV and dK (or dV alone) on the
// second kind of waves, P through LDS too, measured 3-8 us more.  Every sum is the same chain of MFMAs: the same bits.
constexpr int ONCE_NS = 3;
typedef Ring<64, 8, ONCE_NS, true> OnceRing;
typedef Ring<64, 4, 2, false> OnceKeys;   // stage i: rows 64 i .. 64 i + 63 of the group's keys and values
constexpr int ONCE_X = 128 * 64 * 2;      // dS of a block of queries: [128 keys][64 queries], chunks swizzled by aswz
constexpr int ONCE_BYTES = OnceKeys::BYTES + OnceRing::BYTES + 2 * ONCE_X + 4 * OutTile<2>::BYTES;   // ... and outputs' staging

__global__ __launch_bounds__(512, 2) void attn_bwd_once(AttnArgs a, float scale2, float scale) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char asm_[];
  constexpr int D = 64, NKK = 4, NDB = 2, MAXQ = 8;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bi = (a.head0 + blockIdx.y) / a.A, hh = (a.head0 + blockIdx.y) % a.A;
  const long hb = (long)bi * a.s * a.H + hh * D;
  const bf16 *Q = (const bf16*)a.q + hb, *K = (const bf16*)a.k + hb, *V = (const bf16*)a.v + hb, *G = (const bf16*)a.dctx + hb;
  const int nq = a.s / 64, nkg = (a.s + 127) / 128, steps = nkg * nq;   // blocks of queries, groups of keys
  unsigned char *const kv = asm_, *const rg = asm_ + OnceKeys::BYTES, *const xs = rg + OnceRing::BYTES;
  OnceRing ring;
  {
    const float* lse = a.lse + ((long)bi * a.A + hh) * a.s;
    const long T = (long)a.b * a.s;
    const float *d0 = a.delta + ((long)bi * a.A + hh) * a.s, *d1 = nullptr;
    if (a.delta_blocks) {
      d0 = a.delta_blocks + (long)(2 * hh) * T + (long)bi * a.s;
      d1 = d0 + T;
    }
    ring.init(wave < 4 ? Q : G, a.H, a.s, D, wave, lane, [&](int r) { return r == 0 ? lse : (r == 1 ? d0 : (r == 2 ? d1 : nullptr)); });
    ring.m0w += OnceKeys::BYTES;
    ring.m0s += OnceKeys::BYTES;
  }
  // the block of step n + 2, after barrier n (every wave asks for its part of the same blocks, in the same order)
  int asked = 0, asked_q = 0, slot = 0;
  auto ask = [&]() __attribute__((always_inline)) {
    if (asked_q == nq) {
      ring.rewind(a.s);
      asked_q = 0;
    }
    if (asked >= steps) ring.stop();   // past the last one: reads nothing
    ring.request(slot, lane);
    slot = slot + 1 == ONCE_NS ? 0 : slot + 1;
    ++asked;
    ++asked_q;
  };
  // Both kinds of waves pass steps + 1 barriers: step n lies between barriers n and n + 1 for waves 0-3, between n + 1
  // and n + 2 for the others.  KV_LOADS, STORES: requests behind the ring's that a barrier need not wait for.
  typedef OutTile<NDB> Out;
  constexpr int KV_LOADS = 2 * OnceKeys::PER, STORES = 2 * Out::STORES;   // two of the key blocks; dk and dv
  if (wave < 4) {
    for (int i = 0; i < ONCE_NS - 1; ++i) ask();
    int stage = 0, x = 0;
    const int r = 32 * wave + (lane & 31), xr = r * 64 + 4 * h, xsw = aswz<D>(r);   // the lane's key in the group
    for (int g = 0; g < nkg; ++g) {
      const bool live = 128 * g + 32 * wave < a.s;   // (s is a multiple of 64: a wave's keys exist or do not)
      bf16x8 kf[NKK], vf[NKK];
      f32x16 dv[NDB], dk[NDB];  // rows d, column = the lane's key
#pragma unroll
      for (int db = 0; db < NDB; ++db) dv[db] = dk[db] = zero16();
      for (int qb = 0; qb < nq; ++qb) {
        if (g > 0 && qb < 2) OnceRing::wait<STORES>();
        else OnceRing::wait();
        ask();
        if (qb == 0) {
          const bf16* Ks = (const bf16*)(kv + (wave >> 1) * OnceKeys::STAGE);
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) {
            kf[kk] = frag_rows<D>(Ks, (wave & 1) * 32, kk, lane);
            vf[kk] = frag_rows<D>(Ks + OnceKeys::Y_OFF / 2, (wave & 1) * 32, kk, lane);
          }
        }
        const bf16 *Qs = (const bf16*)(rg + stage * OnceRing::STAGE), *Gs = (const bf16*)((const unsigned char*)Qs + OnceRing::Y_OFF);
        const float *Ls = (const float*)((const unsigned char*)Qs + OnceRing::S_OFF), *Ds = Ls + 64;
        bf16* const X = (bf16*)(xs + x * ONCE_X);
        stage = stage + 1 == ONCE_NS ? 0 : stage + 1;
        x ^= 1;
        if (!live) continue;   // (nothing reads these rows of X)
#pragma unroll
        for (int qb2 = 0; qb2 < 2; ++qb2) {
          // every LDS read of a phase before its first MFMA (see attn_fwd_mfma)
          bf16x8 qf[NKK], gf[NKK], gc[2][NDB], qc[2][NDB];
          f32x4 L4[4], D4[4];
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) {
            qf[kk] = frag_rows<D>(Qs, qb2 * 32, kk, lane);
            gf[kk] = frag_rows<D>(Gs, qb2 * 32, kk, lane);
          }
#pragma unroll
          for (int blk = 0; blk < 4; ++blk) {
            const int q = qb2 * 32 + 8 * blk + 4 * h;
            L4[blk] = *(const f32x4*)(Ls + q);
            D4[blk] = *(const f32x4*)(Ds + q) + *(const f32x4*)(Ds + 64 + q);   // (the second block is zero where delta comes whole)
          }
          __builtin_amdgcn_sched_barrier(0);
          f32x16 sa = zero16(), dp = zero16();  // rows: query 32 qb2 + 8 blk + 4 h + e, column: key
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) {
            sa = MFMA(qf[kk], kf[kk], sa);
            dp = MFMA(gf[kk], vf[kk], dp);
          }
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
              gc[ks][db] = frag_cols<D>(Gs, db * 32, qb2 * 32 + ks * 16, lane);
              qc[ks][db] = frag_cols<D>(Qs, db * 32, qb2 * 32 + ks * 16, lane);
            }
          __builtin_amdgcn_sched_barrier(0);
          float p[16], ds[16];
#pragma unroll
          for (int blk = 0; blk < 4; ++blk)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              p[4 * blk + e] = __builtin_amdgcn_exp2f(fmaf(sa[4 * blk + e], scale2, -L4[blk][e]));
              ds[4 * blk + e] = (dp[4 * blk + e] - D4[blk][e]) * p[4 * blk + e];
            }
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 pf = acc_to_operand(p, ks), dsf = acc_to_operand(ds, ks);
            *(bf16x4*)(X + xr + (((4 * qb2 + 2 * ks) ^ xsw) << 3)) = __builtin_shufflevector(dsf, dsf, 0, 1, 2, 3);
            *(bf16x4*)(X + xr + (((4 * qb2 + 2 * ks + 1) ^ xsw) << 3)) = __builtin_shufflevector(dsf, dsf, 4, 5, 6, 7);
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
              dv[db] = MFMA(gc[ks][db], pf, dv[db]);
              dk[db] = MFMA(qc[ks][db], dsf, dk[db]);
            }
          }
        }
      }
      if (g + 1 == nkg) OnceRing::wait();   // (the other waves' last step, not behind these stores)
      if (live) {
        const long o0 = hb + (128L * g + 32 * wave) * a.H;
        float* const S = (float*)(xs + 2 * ONCE_X + wave * Out::BYTES);
        int at = lane;
        asm volatile("" : "+v"(at));   // (addresses made of it are not kept through the loop)
        Out::store(S, dk, scale, (bf16*)a.dk + o0, nullptr, a.H, 32, D, at);
        Out::store(S, dv, 1.f, (bf16*)a.dv + o0, nullptr, a.H, 32, D, at);
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // the last requests (they read nothing) before the wave may end
    return;
  }
  const int w = wave - 4, qt = w & 1, dh = w >> 1;
  OnceKeys keys;
  keys.init(w < 2 ? K : V, a.H, a.s, D, w, lane, [](int) { return (const float*)nullptr; });
  keys.request(0, lane);
  keys.request(1, lane);
  for (int i = 0; i < ONCE_NS - 1; ++i) ask();
  f32x16 dq[MAXQ];   // rows: column 32 dh + 8 blk + 4 h + e of the head, column: query 64 i + 32 qt + (lane & 31)
#pragma unroll
  for (int i = 0; i < MAXQ; ++i) dq[i] = zero16();
  OnceRing::wait();
  ask();
  int x = 0;
  for (int g = 0; g < nkg; ++g) {
    const bool full = 128 * g + 64 < a.s;   // all 128 keys (else the first 64)
    bf16x8 kc[8];
#pragma unroll
    for (int i = 0; i < MAXQ; ++i) {
      if (i < nq) {
        if (i == 2) OnceRing::wait<KV_LOADS>();
        else OnceRing::wait();
        ask();
        if (i == 0) {
#pragma unroll
          for (int p = 0; p < 8; ++p) kc[p] = frag_cols<D>((const bf16*)(kv + p / 4 * OnceKeys::STAGE), dh * 32, p % 4 * 16, lane);
        }
        if (i == 1) {   // every wave has its part of these keys: the next ones (nq >= 4: here before they are needed)
          keys.request(0, lane);
          keys.request(1, lane);
        }
        const bf16* X = (const bf16*)(xs + x * ONCE_X);
        x ^= 1;
        bf16x8 ds[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) ds[p] = frag_cols<D>(X, qt * 32, p * 16, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < 8; ++p)
          if (p < 4 || full) dq[i] = MFMA(kc[p], ds[p], dq[i]);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);
  // (where the keys were: these waves read them last, barriers ago)
  int at = lane;
  asm volatile("" : "+v"(at));   // (addresses made of it are not kept through the loop)
  static_assert(4 * OutTile<1>::BYTES <= OnceKeys::BYTES, "staging of four waves");
#pragma unroll
  for (int i = 0; i < MAXQ; ++i)
    if (i < nq)
      OutTile<1>::store((float*)(kv + w * OutTile<1>::BYTES), &dq[i], scale, (bf16*)a.dq + hb + (64L * i + 32 * qt) * a.H + 32 * dh, nullptr,
                        a.H, 32, 32, at);
}

// ------------------------------------------------------------------ launchers
static bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// Every bf16 head of up to 128 columns in whole 16-byte chunks, at any sequence length
bool attn_uses_mfma(Dtype dt, const AttnArgs& a) {
  return dt == DT_BF16 && a.d % 8 == 0 && a.d <= 128 && a.H % 8 == 0 && (long)a.s * a.H < (1L << 30) - 4096 && al16(a.q) && al16(a.k) && al16(a.v) &&
         al16(a.ctx) && (a.dctx == nullptr || (al16(a.dctx) && al16(a.dq) && al16(a.dk) && al16(a.dv)));
}
bool attn_takes_delta_blocks(Dtype dt, const AttnArgs& a) {
  return attn_uses_mfma(dt, a) && (a.d == 32 || a.d == 64);
}

// f(D, RAG, P32, NW) as constants for the shape: the narrowest block that holds a head; workgroups of four waves (128
// rows), or of two where four would leave a quarter of the 256 units without one (one sample of 512 tokens, 16 heads:
// 64 workgroups of four); roles: workgroups per block of rows (the backward has two)
template <typename F>
static void pick_variant(const AttnArgs& a, int roles, F&& f) {
  typedef std::true_type T;
  typedef std::false_type N;
  const bool rag = a.s % 64 != 0;
  auto waves = [&](auto D, auto RAG, auto P32) {
    if ((long)((a.s + 127) / 128) * a.b * a.A * roles < 192) f(D, RAG, P32, std::integral_constant<int, 2>{});
    else f(D, RAG, P32, std::integral_constant<int, 4>{});
  };
  if (a.d <= 32) {
    if (rag || a.d != 32) waves(std::integral_constant<int, 32>{}, T{}, T{});
    else waves(std::integral_constant<int, 32>{}, N{}, T{});
  } else if (a.d <= 64) {
    if (rag || a.d != 64) waves(std::integral_constant<int, 64>{}, T{}, T{});
    else waves(std::integral_constant<int, 64>{}, N{}, N{});
  } else {
    if (rag || a.d != 128) waves(std::integral_constant<int, 128>{}, T{}, T{});
    else waves(std::integral_constant<int, 128>{}, N{}, T{});
  }
}

hipError_t launch_attn_fwd(Dtype dt, const AttnArgs& a, hipStream_t st) {
  float scale2 = LOG2E / sqrtf((float)a.d);
  if (attn_uses_mfma(dt, a)) {
    hipError_t e = hipSuccess;
    pick_variant(a, 1, [&](auto D, auto RAG, auto P32, auto NW) {
      constexpr int d = decltype(D)::value, nw = decltype(NW)::value, lds = Ring<d, nw, d == 128 ? 2 : 3, false>::BYTES;
      auto kern = attn_fwd_mfma<d, decltype(RAG)::value, decltype(P32)::value, nw>;
      static const hipError_t rc = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if ((e = rc) != hipSuccess) return;
      e = attn_launches(a, [&](const AttnArgs& l, int heads) {
        hipLaunchKernelGGL(kern, dim3((a.s + 32 * nw - 1) / (32 * nw), heads), dim3(64 * nw), lds, st, l, scale2);
        return hipGetLastError();
      });
    });
    return e;
  }
  if (dt == DT_F32 && attn_f32_takes(a)) return launch_attn_fwd_f32(a, st);
  long total = (long)a.b * a.A * a.s * a.d;
  dim3 grid((unsigned)((total + 255) / 256));
  if (dt == DT_BF16) hipLaunchKernelGGL(attn_fwd_plain<bf16>, grid, dim3(256), 0, st, a, scale2);
  else hipLaunchKernelGGL(attn_fwd_plain<float>, grid, dim3(256), 0, st, a, scale2);
  return hipGetLastError();
}

// One workgroup per head, one to a unit, for about three quarters of the time of attn_bwd_mfma's on a full chip (with
// the delta kernel, 512 rows: 256 heads 102 -> 81 us, 192 80 -> 72, 128 53 -> 65; 512 heads of 256 rows 70 -> 57): where
// the turns of the units are three quarters full.  Beside another stream's weight gradients too, although its 152 KB of LDS
// wait for a unit to itself (4 layers each, ms per iteration with attn_bwd_mfma -> so: 768 wide, 192 heads of 256 rows 5.23
// -> 5.21, of 512 10.87 -> 10.86; 640 wide, 200 heads of 320 7.20 -> 7.11; 1024 wide, 256 heads of 256 7.70 -> 7.61, 240 of
// 320 10.13 -> 9.98; 512 wide, 256 of 256 5.71 -> 5.61), and on partitions (four stages of 3 layers on 64 units each, 64
// heads of 512 rows 27.97 -> 27.49).  No bit depends on it.
static bool bwd_once_takes(const AttnArgs& a) {
  const long U = a.units > 0 ? a.units : 256, heads = (long)a.b * a.A;
  return a.d == 64 && a.s % 64 == 0 && a.s >= 256 && a.s <= 512 && 4 * heads >= 3 * U * ((heads + U - 1) / U);
}

hipError_t launch_attn_bwd(Dtype dt, const AttnArgs& a, hipStream_t st) {
  float scale = 1.0f / sqrtf((float)a.d), scale2 = LOG2E * scale;
  const long nd = (long)a.b * a.s * a.A;
  const dim3 gd((unsigned)((nd + 255) / 256));
  hipError_t e;
  if (attn_uses_mfma(dt, a)) {
    if (!a.delta_blocks) {  // no product in front that left delta behind
      const dim3 gr((unsigned)(((long)a.b * a.s + 3) / 4));
      if (a.d == 32) hipLaunchKernelGGL(attn_delta_rows<32>, gr, dim3(256), 0, st, a);
      else if (a.d == 64) hipLaunchKernelGGL(attn_delta_rows<64>, gr, dim3(256), 0, st, a);
      else if (a.d == 128) hipLaunchKernelGGL(attn_delta_rows<128>, gr, dim3(256), 0, st, a);
      else hipLaunchKernelGGL(attn_delta_kernel<bf16>, gd, dim3(256), 0, st, a);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    if (bwd_once_takes(a)) {
      static const hipError_t rc = hipFuncSetAttribute((const void*)attn_bwd_once, hipFuncAttributeMaxDynamicSharedMemorySize, ONCE_BYTES);
      if (rc != hipSuccess) return rc;
      return attn_launches(a, [&](const AttnArgs& l, int heads) {
        hipLaunchKernelGGL(attn_bwd_once, dim3(1, heads), dim3(512), ONCE_BYTES, st, l, scale2, scale);
        return hipGetLastError();
      });
    }
    pick_variant(a, 2, [&](auto D, auto RAG, auto P32, auto NW) {
      constexpr int d = decltype(D)::value, nw = decltype(NW)::value, lds = BwdRing<d, nw>::R::BYTES;
      auto kern = attn_bwd_mfma<d, decltype(RAG)::value, decltype(P32)::value, nw>;
      static const hipError_t rc = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if ((e = rc) != hipSuccess) return;
      e = attn_launches(a, [&](const AttnArgs& l, int heads) {
        hipLaunchKernelGGL(kern, dim3((a.s + 32 * nw - 1) / (32 * nw), heads, 2), dim3(64 * nw), lds, st, l, scale2, scale);
        return hipGetLastError();
      });
    });
    return e;
  }
  if (dt == DT_F32 && attn_f32_takes(a)) return launch_attn_bwd_f32(a, st);
  if (dt == DT_BF16) hipLaunchKernelGGL(attn_delta_kernel<bf16>, gd, dim3(256), 0, st, a);
  else hipLaunchKernelGGL(attn_delta_kernel<float>, gd, dim3(256), 0, st, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  long total = (long)a.b * a.A * a.s * a.d;
  dim3 grid((unsigned)((total + 255) / 256));
  for (int which = 0; which < 3; ++which) {
    if (dt == DT_BF16) hipLaunchKernelGGL(attn_bwd_plain<bf16>, grid, dim3(256), 0, st, a, scale2, scale, which);
    else hipLaunchKernelGGL(attn_bwd_plain<float>, grid, dim3(256), 0, st, a, scale2, scale, which);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dapple
