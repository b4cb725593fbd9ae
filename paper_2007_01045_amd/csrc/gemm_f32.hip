// fp32 products on the fp32 matrix instructions: exact fp32 multiply-adds, fp32 accumulation.
//
// v_mfma_f32_32x32x2_f32 / 16x16x4_f32 do 256 flops per clock and compute unit (157 TFLOP/s for the chip), a
// sixteenth of the bf16 rate, so operand delivery is never the wall here: LDS and the vector caches are used far
// below their rates, and the kernels are bound by the matrix pipe once every SIMD has a wave.  What decides the time
// is therefore how many SIMDs a product reaches:
//  * gemm_f32_kernel<128> / <64>: a square tile per workgroup of 2x2 waves, 32-wide k-tiles through a double buffer
//    in LDS (2 x 37 KB: two workgroups per unit), the next two tiles' global loads in flight behind the MFMAs;
//  * gemm_f32_small<TW>: 16 TW square tiles, one per workgroup whose four waves take every fourth 16-wide piece of K
//    straight from global memory and add their partial tiles in wave order through LDS: for products with so few
//    tiles that the length of one wave's MFMA chain, or the launch's memory latencies, are the time (32 x 64 x 64 with
//    both operands' loads unmasked and a wave's pieces of K counted in scalar registers: 4.6 -> 2.9 us);
//  * gemm_f32_quad: the sums of gemm_f32_small in the 64-wide tiles of gemm_f32_kernel, every wave with four sets of
//    accumulators: for a group of micro-batches of which one alone takes the small kernel.
// Measured before -> after: 2 layers of 1024 x 4096, 2 x 512 tokens, 2 micro-batches: 412 -> 3.3 ms per iteration
// with the attention kernels of attention_f32.hip (one thread per output element before).
#include <type_traits>
#include <utility>

#include "device_common.h"
#include "gemm_epilogue.h"
#include "kernels.h"
#include "reduce_jobs.h"

namespace dapple {

// ------------------------------------------------------------------ LDS-tiled kernel
constexpr int FBK = 32;

// One operand's [R x 32] k-tile.  k-contiguous: LDS [R][32 + 4]; 16 lanes reading 16 rows 16 bytes each hit all 64
// banks.  k-strided: LDS [32][R + 8]; the two half waves of a 4-byte read lie 4 rows = 32 banks apart.
// Loads carry no condition: rows past the end and, in a segment's last tile, k entries past its end re-read the last
// ones, and are zeroed on their way to LDS.
// (BK = 64, for 16-row fragments: LDS [64][R + 4] there, the four lane groups of a 4-byte read lie 4 rows = 16 banks
// apart.)
template <int R, bool KS, int BK = FBK>
struct F32Tile {
  static constexpr int LD = KS ? R + (BK == 64 ? 4 : 8) : BK + 4;
  static constexpr int FLOATS = KS ? BK * LD : R * LD;
  static constexpr int N = R * BK / 4 / 256;   // float4 per thread
  f32x4 v[N];
  unsigned off[N], off_tail[N];   // bytes from the tile's first element; of a segment's last tile
  bool tail;                      // v holds a segment's last tile
  int tail_k;                     // ... which has this many k entries
  unsigned live;                  // bit i: piece i lies inside the operand's rows
  static __device__ __forceinline__ int row_of(int pos) { return KS ? pos % (R / 4) * 4 : pos / (BK / 4); }
  static __device__ __forceinline__ int k_of(int pos) { return KS ? pos / (R / 4) : pos % (BK / 4) * 4; }
  // rows: valid rows from the tile's first one on
  __device__ __forceinline__ void init(int ld, int rows, int tk, int tid) {
    tail_k = tk;
    live = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int pos = tid + 256 * i, r = KS ? min(row_of(pos), (rows - 1) & ~3) : min(row_of(pos), rows - 1);
      const int k = k_of(pos), kt = min(k, KS ? tk - 1 : (tk - 1) & ~3);
      live |= row_of(pos) < rows ? 1u << i : 0u;
      off[i] = 4u * (unsigned)(KS ? k * ld + r : r * ld + k);
      off_tail[i] = 4u * (unsigned)(KS ? kt * ld + r : r * ld + kt);
    }
  }
  // next: first element of the tile
  __device__ __forceinline__ void load(const char* next, bool is_tail) {
    tail = is_tail;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = *(const f32x4*)(next + (is_tail ? off_tail[i] : off[i]));
  }
  __device__ __forceinline__ void store(float* S, int tid) const {
    const int valid = tail ? tail_k : BK;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int pos = tid + 256 * i;
      const int a = KS ? k_of(pos) : row_of(pos), b = KS ? row_of(pos) : k_of(pos);
      const bool in = k_of(pos) < valid && (live >> i & 1);
      f32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = in ? v[i][e] : 0.f;
      *(f32x4*)(S + a * LD + b) = x;
    }
  }
  // row r, k = 8 kk + 4 h + 0..3
  static __device__ __forceinline__ f32x4 frag(const float* S, int r, int kk, int h) {
    const int k = 8 * kk + 4 * h;
    if (!KS) return *(const f32x4*)(S + r * LD + k);
    return f32x4{S[k * LD + r], S[(k + 1) * LD + r], S[(k + 2) * LD + r], S[(k + 3) * LD + r]};
  }
  // row r, k = 16 piece + 4 q4 + 0..3
  static __device__ __forceinline__ f32x4 frag16(const float* S, int r, int piece, int q4) { return frag(S, r, 2 * piece, q4); }
};

// The tiles of both operands, in order: two sets of registers, so that a tile is requested two k-tiles before it is used.
// (With one set it was a k-tile's time, about what memory takes: 2048 x 1024 x 4096 in 64-wide tiles 184 -> 146 us, the
// 128-wide tile 3%.)
template <bool AKS, bool BKS, typename TA, typename TB, int BK>
struct F32Feed {
  struct Set {
    TA a;
    TB b;
  };
  static constexpr int STAGE = TA::FLOATS + TB::FLOATS;
  Set s0, s1;
  const char *a_next, *b_next;   // first elements of the next tile
  long a_step, b_step, a_jump, b_jump;
  int per_seg, kt, left;         // tiles per segment; the next one's place in its segment; tiles not yet requested
  __device__ __forceinline__ void init(const GemmArgs& g, int z, int m0, int n0, int klen, int tid) {
    per_seg = (klen + BK - 1) / BK;
    left = g.K / g.kseg_len * per_seg;
    kt = 0;
    const int tail_k = klen - (per_seg - 1) * BK;
    s0.a.init(g.lda, g.m_valid - m0, tail_k, tid);
    s0.b.init(g.ldb, g.n_valid - n0, tail_k, tid);
    s1 = s0;
    a_next = (const char*)((const float*)g.A + z * g.sA + (AKS ? (long)m0 : (long)m0 * g.lda));
    b_next = (const char*)((const float*)g.B + z * g.sB + (BKS ? (long)n0 : (long)n0 * g.ldb));
    a_step = 4L * BK * (AKS ? g.lda : 1);
    b_step = 4L * BK * (BKS ? g.ldb : 1);
    a_jump = 4L * g.segA - (per_seg - 1) * a_step;
    b_jump = 4L * g.segB - (per_seg - 1) * b_step;
  }
  __device__ __forceinline__ void load(Set& s) {   // the next tile; past the last one that one again
    s.a.load(a_next, kt == per_seg - 1);
    s.b.load(b_next, kt == per_seg - 1);
    --left;
    const bool last = kt == per_seg - 1, more = left > 0;
    a_next += more ? (last ? a_jump : a_step) : 0;
    b_next += more ? (last ? b_jump : b_step) : 0;
    kt = more ? (last ? 0 : kt + 1) : kt;
  }
  static __device__ __forceinline__ void store(const Set& s, float* S, int tid) {
    s.a.store(S, tid);
    s.b.store(S + TA::FLOATS, tid);
  }
  // f(now, then) for every k-tile: its operands are in LDS, `now` is to take the tile after the next one, `then` holds
  // the next one
  template <typename F>
  __device__ __forceinline__ void each(int tiles, F&& f) {
    for (; tiles > 1; tiles -= 2) {
      f(s0, s1);
      f(s1, s0);
    }
    if (tiles) {
      f(s0, s1);
      const Set x = s0;   // the sets change places
      s0 = s1;
      s1 = x;
    }
  }
};

// CS: the variant that can also sum B over k (EPI_BSUM).  The k-loop holds no branch: one had the accumulators copied
// between the register files in every k-tile (2048 x 1024 x 4096: 190 us with it).
template <int BT, bool AKS, bool BKS, bool CS>
__device__ __forceinline__ void f32_tile(const GemmArgs& g, int tiles_m, int tiles_n, const int bid, const int z) {
  typedef F32Tile<BT, AKS> TA;
  typedef F32Tile<BT, BKS> TB;
  constexpr int W = BT / 2, NB = W / 32;   // wave tile, 32-blocks per side
  extern __shared__ __attribute__((aligned(16))) float fsm[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l31 = lane & 31, h = lane >> 5;
  int tm, tn;
  tile_of(bid, tiles_m, tiles_n, BT, BT, tm, tn);
  const int m0 = tm * BT, n0 = tn * BT, wm0 = (wave >> 1) * W, wn0 = (wave & 1) * W;
  float* const bs = CS && (g.epi & EPI_BSUM) && z == 0 ? g.bsum : nullptr;
  const bool do_cs = bs != nullptr && tm == 0 && wm0 == 0;
  const int klen = g.K > g.kseg_len ? g.kseg_len : min(g.K, g.k_valid);
  const int per_seg = (klen + FBK - 1) / FBK, nseg = g.K / g.kseg_len;
  f32x16 acc[NB][NB];
  float cs[NB];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      cs[i] = 0.f;
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    }
  };
  clear();
  typedef F32Feed<AKS, BKS, TA, TB, FBK> Feed;
  Feed feed;
  feed.init(g, z, m0, n0, klen, tid);
  feed.load(feed.s0);
  feed.load(feed.s1);
  Feed::store(feed.s0, fsm, tid);
  __syncthreads();
  const long zc = z * g.sC, zb = z * g.sBias;
  auto finish = [&]() __attribute__((always_inline)) {   // add the column sums and store the tile
    if (CS && do_cs) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const float t = cs[j] + __shfl_xor(cs[j], 32, 64);
        const int col = n0 + wn0 + 32 * j + l31;
        if (h == 0 && col < g.N) bs[col] += t;
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int row = m0 + wm0 + 32 * i + l31;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        // what a 32x32 block's epilogue reads, all of it before its first store: behind a store to the same matrix the
        // compiler leaves a load where it stands, one trip to memory after the other
        Epilogue4 in[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = n0 + wn0 + 32 * j + 8 * q + 4 * h;
          in[q] = row < g.M && col < g.N ? epilogue_load4(g, zc, zb, row, col) : Epilogue4{};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int col = n0 + wn0 + 32 * j + 8 * q + 4 * h;
          if (row < g.M && col < g.N)
            epilogue_store4(g, zc, row, col,
                            f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]}, in[q]);
        }
      }
    }
  };
  int buf = 0;
  auto k_tile = [&](typename Feed::Set& now, const typename Feed::Set& then, auto WCS) __attribute__((always_inline)) {
    const float *SA = fsm + buf * Feed::STAGE, *SB = SA + TA::FLOATS;
    feed.load(now);
    __builtin_amdgcn_sched_barrier(0);   // (the loads would sink to their use, behind the products that cover them)
#pragma unroll
    for (int kk = 0; kk < FBK / 8; ++kk) {
      f32x4 a[NB], b[NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) a[i] = TA::frag(SA, wm0 + 32 * i + l31, kk, h);
#pragma unroll
      for (int j = 0; j < NB; ++j) b[j] = TB::frag(SB, wn0 + 32 * j + l31, kk, h);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j)   // B first: a lane then owns 4 consecutive columns of one row
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j][e], a[i][e], acc[i][j], 0, 0, 0);
      if constexpr (decltype(WCS)::value) {
#pragma unroll
        for (int j = 0; j < NB; ++j) cs[j] += (b[j][0] + b[j][1]) + (b[j][2] + b[j][3]);
      }
    }
    buf ^= 1;
    Feed::store(then, fsm + buf * Feed::STAGE, tid);
    __syncthreads();
  };
  auto k_loop = [&](int tiles, auto WCS) __attribute__((always_inline)) {
    feed.each(tiles, [&](typename Feed::Set& now, const typename Feed::Set& then) __attribute__((always_inline)) { k_tile(now, then, WCS); });
  };
  // EPI_SEGACC: a segment's sum goes to C on its own
  const bool segacc = (g.epi & EPI_SEGACC) != 0;
  const int turns = segacc ? nseg : 1, tiles = segacc ? per_seg : nseg * per_seg;
  for (int s = 0; s < turns; ++s) {
    if (s) clear();
    if constexpr (CS) {
      if (do_cs) k_loop(tiles, std::true_type{});
      else k_loop(tiles, std::false_type{});
    } else {
      k_loop(tiles, std::false_type{});
    }
    finish();
  }
}

// ------------------------------------------------------------------ few tiles: K split over the waves
// (NSG = 2: accumulating products over an even number of segments, two of them in flight together)
template <int TW, bool AKS, bool BKS, int NSG = 1>
__device__ __forceinline__ void f32_small_tile(GemmArgs g, int tiles_n, const int bid, const int z) {
  constexpr int BT = 16 * TW, LD = BT + 4;
  __shared__ __attribute__((aligned(16))) float part[NSG][4][BT * LD];
  __shared__ float cpart[NSG][4][BT];
  const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, q4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (uniform: a wave's pieces of K are counted in scalar registers)
  const int tm = bid / tiles_n, tn = bid % tiles_n;
  const int m0 = tm * BT, n0 = tn * BT;
  const float *A = (const float*)g.A + z * g.sA, *B = (const float*)g.B + z * g.sB;
  float* const bs = (g.epi & EPI_BSUM) && z == 0 ? g.bsum : nullptr;
  const int klen = g.K > g.kseg_len ? g.kseg_len : min(g.K, g.k_valid);
  const int per_seg = (g.kseg_len + 15) / 16, nseg = g.K / g.kseg_len;
  // EPI_SEGACC: the segments one after the other, NSG of them at a time, each one's sum added to C; else all of them
  // as one sum
  const bool segacc = (g.epi & EPI_SEGACC) != 0;
  const int nc = segacc ? per_seg : nseg * per_seg;
  const long zc = z * g.sC, zb = z * g.sBias;
  // the part of the tile a thread stores (at most one piece of four columns), and what its epilogue reads: requested
  // first of all, a launch this small is little else than memory latencies in a row
  const int er = tid * 4 / BT, ec = tid * 4 % BT, row = m0 + er, col = n0 + ec;
  const bool stores = tid * 4 < BT * BT && row < g.M && col < g.N;
  const bool sums = bs && tm == 0 && tid < BT && n0 + tid < g.N;
  for (int turn = 0; turn < (segacc ? nseg : 1); turn += NSG, A += NSG * g.segA, B += NSG * g.segB) {
    const Epilogue4 in = stores ? epilogue_load4(g, zc, zb, row, col) : Epilogue4{};
    float bsum0 = sums ? bs[n0 + tid] : 0.f;
    f32x4 acc[NSG][TW][TW];
    float cs[NSG][TW];
#pragma unroll
    for (int s = 0; s < NSG; ++s)
#pragma unroll
      for (int i = 0; i < TW; ++i) {
        cs[s][i] = 0.f;
#pragma unroll
        for (int j = 0; j < TW; ++j) acc[s][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    // rows l15 of the 16-row block at r0, k = k0 + 4 q4 + 0..3.  No branch: what lies outside re-reads the last row or k,
    // and is zeroed before it is used (a launch this small is latencies in a row, a masked load a branch of its own).
    auto fetch = [&](const float* X, int ld, bool ks, int r, int rows, int k0) __attribute__((always_inline)) {
      const int k = k0 + 4 * q4, rr = min(r, rows - 1);
      if (!ks) return *(const f32x4*)(X + (long)rr * ld + min(k, (klen - 1) & ~3));
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = X[(long)min(k + e, klen - 1) * ld + rr];
      return v;
    };
    auto inside = [&](f32x4& v, bool ks, int r, int rows, int k0) __attribute__((always_inline)) {
      const int k = k0 + 4 * q4;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = r < rows && (ks ? k + e : k) < klen ? v[e] : 0.f;
    };
    // segment and first k of piece c
    auto piece = [&](int c, int& seg, int& k0) __attribute__((always_inline)) {
      seg = 0;
      k0 = 16 * c;
      if (NSG == 1 && !segacc && nseg > 1) {   // (an integer division: only where there are segments)
        seg = c / per_seg;
        k0 -= seg * per_seg * 16;
      }
    };
    constexpr int U = (TW == 1 ? 8 : 4) / NSG;   // 16-wide pieces of K (of each segment) whose loads are in flight together
    for (int c0 = wave; c0 < nc; c0 += 4 * U) {
      f32x4 a[NSG][U][TW], b[NSG][U][TW];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + 4 * u;
        if (c >= nc) break;
        int seg, k0;
        piece(c, seg, k0);
#pragma unroll
        for (int s = 0; s < NSG; ++s) {
          const float *As = A + (NSG > 1 ? s : seg) * g.segA, *Bs = B + (NSG > 1 ? s : seg) * g.segB;
#pragma unroll
          for (int i = 0; i < TW; ++i) {
            a[s][u][i] = fetch(As, g.lda, AKS, m0 + 16 * i + l15, g.m_valid, k0);
            b[s][u][i] = fetch(Bs, g.ldb, BKS, n0 + 16 * i + l15, g.n_valid, k0);
          }
        }
      }
#pragma unroll
      for (int s = 0; s < NSG; ++s)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (c0 + 4 * u >= nc) break;
          int seg, k0;
          piece(c0 + 4 * u, seg, k0);
#pragma unroll
          for (int i = 0; i < TW; ++i) {
            inside(a[s][u][i], AKS, m0 + 16 * i + l15, g.m_valid, k0);
            inside(b[s][u][i], BKS, n0 + 16 * i + l15, g.n_valid, k0);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TW; ++i)
#pragma unroll
              for (int j = 0; j < TW; ++j)
                acc[s][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[s][u][j][e], a[s][u][i][e], acc[s][i][j], 0, 0, 0);
          if (bs) {
#pragma unroll
            for (int j = 0; j < TW; ++j) cs[s][j] += (b[s][u][j][0] + b[s][u][j][1]) + (b[s][u][j][2] + b[s][u][j][3]);
          }
        }
    }
    if (turn) __syncthreads();   // the partial tiles of the segments before have been read
    // acc[s][i][j]: row 16 i + l15, columns 16 j + 4 q4 + 0..3
#pragma unroll
    for (int s = 0; s < NSG; ++s) {
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j) *(f32x4*)(part[s][wave] + (16 * i + l15) * LD + 16 * j + 4 * q4) = acc[s][i][j];
      if (bs && tm == 0) {
#pragma unroll
        for (int j = 0; j < TW; ++j) {
          float t = cs[s][j];
          t += __shfl_xor(t, 16, 64);
          t += __shfl_xor(t, 32, 64);
          if (q4 == 0) cpart[s][wave][16 * j + l15] = t;
        }
      }
    }
    __syncthreads();
    if (sums) {
#pragma unroll
      for (int s = 0; s < NSG; ++s) bsum0 += ((cpart[s][0][tid] + cpart[s][1][tid]) + cpart[s][2][tid]) + cpart[s][3][tid];
      bs[n0 + tid] = bsum0;
    }
    if (!stores) continue;
    auto sum_of = [&](int s) {
      const int o = er * LD + ec;
      const f32x4 p0 = *(const f32x4*)(part[s][0] + o), p1 = *(const f32x4*)(part[s][1] + o), p2 = *(const f32x4*)(part[s][2] + o),
                  p3 = *(const f32x4*)(part[s][3] + o);
      return ((p0 + p1) + p2) + p3;
    };
    if constexpr (NSG == 2) {   // an accumulating product
      *(f32x4*)((float*)g.C + zc + (long)row * g.ldc + col) = (in.c + sum_of(0)) + sum_of(1);
    } else {
      epilogue_store4(g, zc, row, col, sum_of(0), in);
    }
  }
}

// ------------------------------------------------------------------ the small kernel's sums in large tiles
// A group of micro-batches has rows enough for 64-wide tiles where one of them has not, but must add as one does (see
// launch_layout): every wave of a 64x64 tile keeps the four chains of f32_small_tile, piece c of K in set c % 4, for
// its 32x32 part (64 accumulator registers) and adds the sets in the same order.  k-tiles of 64 so that a piece's set
// is a constant; a segment's last one may be short only where there is one segment (the pieces are counted through).
// 8 micro-batches of 256 rows, 512 wide, GPipe order: 1.51 ms with the small kernel's 32-wide tiles, 1.13 so.
template <bool BKS>
__device__ __forceinline__ void f32_quad_tile(const GemmArgs& g, int tiles_m, int tiles_n, const int bid, const int z) {
  constexpr int BK = 64;
  typedef F32Tile<64, false, BK> TA;
  typedef F32Tile<64, BKS, BK> TB;
  extern __shared__ __attribute__((aligned(16))) float fsm[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l15 = lane & 15, q4 = lane >> 4;
  int tm, tn;
  tile_of(bid, tiles_m, tiles_n, 64, 64, tm, tn);
  const int m0 = tm * 64, n0 = tn * 64, wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
  const int klen = g.K > g.kseg_len ? g.kseg_len : min(g.K, g.k_valid);
  f32x4 acc[4][2][2];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[c][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  typedef F32Feed<false, BKS, TA, TB, BK> Feed;
  Feed feed;
  feed.init(g, z, m0, n0, klen, tid);
  const int tiles = feed.left;
  feed.load(feed.s0);
  feed.load(feed.s1);
  Feed::store(feed.s0, fsm, tid);
  __syncthreads();
  int buf = 0;
  feed.each(tiles, [&](typename Feed::Set& now, const typename Feed::Set& then) __attribute__((always_inline)) {
    const float *SA = fsm + buf * Feed::STAGE, *SB = SA + TA::FLOATS;
    feed.load(now);
    __builtin_amdgcn_sched_barrier(0);   // (see f32_tile)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      f32x4 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = TA::frag16(SA, wm0 + 16 * i + l15, c, q4);
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = TB::frag16(SB, wn0 + 16 * j + l15, c, q4);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[c][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][e], a[i][e], acc[c][i][j], 0, 0, 0);
    }
    buf ^= 1;
    Feed::store(then, fsm + buf * Feed::STAGE, tid);
    __syncthreads();
  });
  const long zc = z * g.sC, zb = z * g.sBias;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = m0 + wm0 + 16 * i + l15;
    Epilogue4 in[2];   // all reads before the first store (see f32_tile)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + wn0 + 16 * j + 4 * q4;
      in[j] = row < g.M && col < g.N ? epilogue_load4(g, zc, zb, row, col) : Epilogue4{};
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + wn0 + 16 * j + 4 * q4;
      if (row < g.M && col < g.N)
        epilogue_store4(g, zc, row, col, ((acc[0][i][j] + acc[1][i][j]) + acc[2][i][j]) + acc[3][i][j], in[j]);
    }
  }
}

// ------------------------------------------------------------------ kernels
template <bool BKS>
__global__ __launch_bounds__(256, 2) void gemm_f32_quad(GemmArgs g, int tiles_m, int tiles_n) {
  f32_quad_tile<BKS>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.z);
}
template <int BT, bool AKS, bool BKS>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  f32_tile<BT, AKS, BKS, AKS && BKS>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.z);
}
template <int TW, bool AKS, bool BKS>
__global__ __launch_bounds__(256) void gemm_f32_small(GemmArgs g, int tiles_n) {
  f32_small_tile<TW, AKS, BKS>(g, tiles_n, blockIdx.x, blockIdx.z);
}

// a list of weight-gradient products in one launch (first[k]: first workgroup of problem k); BT = 128, 64: the tile
// kernel, 32, 16: the small one
struct F32Tiles {
  int first[WgradGroup::MAX + 1];
};
template <int BT, int NSG>
__global__ __launch_bounds__(256, 2) void wgrad_group_f32(WgradGroup w, F32Tiles t) {
  if ((int)blockIdx.x >= t.first[w.n]) {   // behind the products' tiles: the sums
    __shared__ float red[4][64];
    const int b = blockIdx.x - t.first[w.n], per = (w.jobs.j[0].cols + 63) / 64;
    reduce_columns(w.jobs.j[b / per], w.jobs.nmb, w.jobs.mb_stride, b % per, 1, red);
    return;
  }
  int i = 0;
#pragma unroll
  for (int k = 1; k < WgradGroup::MAX; ++k) i += k < w.n && (int)blockIdx.x >= t.first[k];
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
  g.epi = EPI_ACC32 | (g.bsum ? EPI_BSUM : 0) | (w.K > w.kseg ? EPI_SEGACC : 0);
  const int tn = (g.N + BT - 1) / BT, bid = blockIdx.x - first;
  if constexpr (BT >= 64) f32_tile<BT, true, true, true>(g, (g.M + BT - 1) / BT, tn, bid, 0);
  else f32_small_tile<BT / 16, true, true, NSG>(g, tn, bid, 0);
}

// ------------------------------------------------------------------ host side
static bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

bool gemm_f32_takes(const GemmArgs& g) {
  if (g.K < 1 || g.kseg_len < 1 || g.K % g.kseg_len || g.N % 4 || g.lda % 4 || g.ldb % 4 || g.ldc % 4) return false;
  if (g.kseg_len % 4 && !(g.a_kstrided && g.b_kstrided)) return false;
  if (g.sA % 4 || g.sB % 4 || g.sC % 4 || g.sBias % 4 || g.segA % 4 || g.segB % 4) return false;
  if (!al16(g.A) || !al16(g.B) || !al16(g.C) || (g.epi & (EPI_ROWDOT | EPI_AUXLN))) return false;
  // a k-strided operand is read four rows' entries at a time: what lies past the last row must be the padding of its
  // leading dimension, and must not reach a stored element
  if (g.a_kstrided && g.m_valid % 4 && (g.m_valid != g.M || (g.m_valid + 3) / 4 * 4 > g.lda)) return false;
  if (g.b_kstrided && g.n_valid % 4) return false;
  if (!g.a_kstrided && !g.b_kstrided && g.k_valid < g.K) return false;   // k_valid cuts k-strided operands
  // no tile begins past the last row
  if (g.M > (g.m_valid + 63) / 64 * 64 || g.N > (g.n_valid + 63) / 64 * 64) return false;
  if ((g.epi & EPI_BIAS) && !al16(g.bias)) return false;
  if ((g.epi & (EPI_ADD | EPI_MUL)) && (g.ldaux % 4 || !al16(g.aux))) return false;
  if ((g.epi & EPI_GELU) && !al16(g.C2)) return false;
  if ((g.epi & EPI_BSUM) && !(g.a_kstrided && g.b_kstrided)) return false;
  return true;
}

template <int BT, bool AKS, bool BKS>
static hipError_t launch_tile(const GemmArgs& g, hipStream_t st) {
  auto kern = gemm_f32_kernel<BT, AKS, BKS>;
  constexpr int lds = 2 * 4 * (F32Tile<BT, AKS>::FLOATS + F32Tile<BT, BKS>::FLOATS);
  static const hipError_t attr_rc = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr_rc != hipSuccess) return attr_rc;
  const int tm = (g.M + BT - 1) / BT, tn = (g.N + BT - 1) / BT;
  hipLaunchKernelGGL(kern, dim3(tm * tn, 1, g.batch), dim3(256), lds, st, g, tm, tn);
  return hipGetLastError();
}
template <bool BKS>
static hipError_t launch_quad(const GemmArgs& g, hipStream_t st) {
  auto kern = gemm_f32_quad<BKS>;
  constexpr int lds = 2 * 4 * (F32Tile<64, false, 64>::FLOATS + F32Tile<64, BKS, 64>::FLOATS);
  static const hipError_t attr_rc = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (attr_rc != hipSuccess) return attr_rc;
  const int tm = (g.M + 63) / 64, tn = (g.N + 63) / 64;
  hipLaunchKernelGGL(kern, dim3(tm * tn, 1, g.batch), dim3(256), lds, st, g, tm, tn);
  return hipGetLastError();
}
template <int TW, bool AKS, bool BKS>
static hipError_t launch_small(const GemmArgs& g, hipStream_t st) {
  const int tm = (g.M + 16 * TW - 1) / (16 * TW), tn = (g.N + 16 * TW - 1) / (16 * TW);
  hipLaunchKernelGGL((gemm_f32_small<TW, AKS, BKS>), dim3(tm * tn, 1, g.batch), dim3(256), 0, st, g, tn);
  return hipGetLastError();
}

// 128-wide tiles rather than 64-wide ones: where there are enough for most of the 256 units (a stream with fewer of them has
// the same line) and the fullest of its units has no more work than with the 64-wide ones' finer split (three products of 2048 x 1024 x 1024, 384 tiles: 143 -> 112 us)
static bool large_tiles(long t128, long t64, int units) {
  const long U = units > 0 ? units : 256;
  return t128 >= 192 && 40 * ((t128 + U - 1) / U) <= 11 * ((t64 + U - 1) / U);
}

template <bool AKS, bool BKS>
static hipError_t launch_layout(const GemmArgs& g, hipStream_t st) {
  auto tiles_of = [&](long rows, long t) { return ((rows + t - 1) / t) * ((g.N + t - 1) / t) * g.batch; };
  auto tiles = [&](long t) { return tiles_of(g.M, t); };
  // Two orders of summation: one ascending chain (the tile kernel), and four waves' chains added up (the small one).
  // Which of them follows from the rows of ONE micro-batch; the tile inside an order, which no bit depends on, from all
  // the rows.  The largest tile that still gives most of the 256 units a workgroup.  Below that the 32- and 16-wide tiles
  // with K split over the waves: a 16-wide one has a quarter of the MFMA chain but reads every operand element twice as
  // often.
  const bool chain = tiles_of(g.rows1 > 0 ? g.rows1 : g.M, 64) >= 160;
  if (chain) return large_tiles(tiles(128), tiles(64), g.units) ? launch_tile<128, AKS, BKS>(g, st) : launch_tile<64, AKS, BKS>(g, st);
  if constexpr (!AKS)
    if (tiles(64) >= 160 && !(g.epi & EPI_SEGACC) && (g.K == g.kseg_len || g.kseg_len % 64 == 0)) return launch_quad<BKS>(g, st);
  if (tiles(32) >= 160) return launch_small<2, AKS, BKS>(g, st);
  return launch_small<1, AKS, BKS>(g, st);
}

template <int BT, int NSG>
static hipError_t launch_group_of(const WgradGroup& w, hipStream_t st) {
  auto kern = wgrad_group_f32<BT, NSG>;
  int lds = 0;
  if constexpr (BT >= 64) {
    constexpr int bytes = 2 * 4 * 2 * F32Tile<BT, true>::FLOATS;
    static const hipError_t attr_rc = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (attr_rc != hipSuccess) return attr_rc;
    lds = bytes;
  }
  F32Tiles t{};
  for (int i = 0; i < w.n; ++i) t.first[i + 1] = t.first[i] + ((w.p[i].M + BT - 1) / BT) * ((w.p[i].N + BT - 1) / BT);
  hipLaunchKernelGGL(kern, dim3(t.first[w.n] + w.job_blocks()), dim3(256), lds, st, w, t);
  return hipGetLastError();
}

template <int BT>
static hipError_t launch_group(const WgradGroup& w, hipStream_t st) {
  if constexpr (BT < 64)   // (the tile kernel takes the segments one after the other)
    if (w.K / w.kseg % 2 == 0) return launch_group_of<BT, 2>(w, st);
  return launch_group_of<BT, 1>(w, st);
}

hipError_t launch_wgrad_group_f32(const WgradGroup& w, hipStream_t st) {
  auto tiles = [&](long b) {
    long n = 0;
    for (int i = 0; i < w.n; ++i) n += ((w.p[i].M + b - 1) / b) * ((w.p[i].N + b - 1) / b);
    return n;
  };
  if ((w.list_tiles64 > 0 ? w.list_tiles64 : tiles(64)) >= 160)   // the lines of launch_layout
    return large_tiles(tiles(128), tiles(64), w.units) ? launch_group<128>(w, st) : launch_group<64>(w, st);
  if (tiles(32) >= 160) return launch_group<32>(w, st);
  return launch_group<16>(w, st);
}

hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t st) {
  if (g.a_kstrided) return g.b_kstrided ? launch_layout<true, true>(g, st) : launch_layout<true, false>(g, st);
  return g.b_kstrided ? launch_layout<false, true>(g, st) : launch_layout<false, false>(g, st);
}

}  // namespace dapple
