// The bf16 MFMA product kernel (see gemm.hip for the outline): a template over the workgroup's tile, its waves, the LDS
// ring and the operand layouts.  Instantiated per layout in gemm_nn.hip, gemm_nt.hip, gemm_tn.hip and gemm_tt.hip.
#pragma once
#include <type_traits>
#include <utility>

#include "device_common.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace dapple {

constexpr unsigned BUF_RSRC_FLAGS = 0x00020000;  // raw buffer, 32-bit data format (gfx9 family)

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int int4v;

// One operand's [R x BK] tile of a k-step in LDS (BK = 64 or 32), filled by buffer loads that
// write straight into LDS (16 bytes per lane, 1 KiB contiguous per wave
// instruction; out-of-range offsets read as zero, so ragged edges need no
// branches) and read back as MFMA fragments.
//   k-contiguous operand: LDS [row][BK/8 chunks of 16 B], chunk' = chunk ^ rswz(row)
//                         (BK = 64: (row >> 1) & 7; BK = 32: (row >> 2) & 3 -- in both cases the 16 rows a
//                         group of 16 lanes reads spread over all 16 sixteen-byte slots of a 256-byte bank row)
//   k-strided operand:    LDS [k][R/8 chunks],         chunk' = chunk ^ kswz(k)
// LDS has 64 banks of 4 bytes: a 128-bit read is served 16 lanes at a time and a
// 64-bit (transpose) read 32 lanes at a time, each group needing 256 distinct
// bytes modulo 256.  The swizzles give exactly that (measured: 5 and 2.6 clocks
// per wave instruction against 8 and 8 unswizzled); they are applied on the global
// side (which chunk a lane fetches), since the LDS side of a direct load is fixed
// to lane order.
//
// A wave issues one instruction every few clocks, and a k-step of a 64x64 wave tile is
// only 16 MFMAs: the loop is bound by instruction issue unless everything around the
// MFMAs is a handful of instructions.  So every per-lane address is computed once,
// before the loop (global side: voff; LDS side: FragAddr), the ring slot enters as an
// instruction immediate (the k-loop is unrolled over the ring), and the global cursor
// is a buffer resource in scalar registers that advances by two scalar adds per k-step.
template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop whose index is a constant expression
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// KT: the last k-tile of a K segment may be short (a multiple of 8).  A k-strided operand needs nothing for that:
// its rows beyond the segment lie beyond the buffer's record count and read as zero.  A k-contiguous one would
// read on into its next row; there the lanes whose 16-byte chunk lies beyond the segment are given an offset
// outside the buffer for that one tile (a select per load and k-tile, in the shadow of the MFMAs).
template <int R, bool KS, int NW, int BK, bool KT = false>
struct OperandTile {
  static_assert(BK == 64 || BK == 32, "k-tiles of 64 or 32");
  static constexpr int CH = BK / 8;                   // 16-byte chunks per row of a k-contiguous tile
  static constexpr int NI = R * CH / (64 * NW);       // load instructions per wave per k-tile
  static constexpr int LDS_ELEMS = R * BK;
  static constexpr int LDS_BYTES = LDS_ELEMS * 2;
  static_assert(R * CH % (64 * NW) == 0, "tile rows must split evenly over the waves");
  int voff[NI];  // per-lane byte offset of each load inside the k-tile's slab
  static constexpr bool MASKED = KT && !KS;
  int vfull[MASKED ? NI : 1];  // the offsets of a whole k-tile, and which of them a short one leaves out
  unsigned over;

  // chunk swizzle of row `row` of a k-contiguous tile
  static __device__ __forceinline__ int rswz(int row) { return BK == 64 ? (row >> 1) & 7 : (row >> 2) & 3; }

  // chunk swizzle of k row k of a k-strided tile: rows of 256 B or more rotate by 64 B per
  // row (4 rows cover 256 B); rows of 128 B alternate halves every second row; four rows of 64 B are 256 B as they are
  static __device__ __forceinline__ int kswz(int k) { return R >= 128 ? (k & 3) << 2 : R == 64 ? ((k >> 1) & 1) << 2 : 0; }

  // A wave loads NI consecutive 1 KiB chunks of the tile.  The instruction's immediate offset is
  // added to the global AND to the LDS address, so the loads of a group of up to four chunks share
  // one M0 (the LDS base) and differ in the immediate; the lane offsets are compensated
  // (voff_j - 1024 j) and, to stay non-negative, shifted by BIAS, which the kernel takes out of
  // the buffer's base and adds to its record count.
  static constexpr int BIAS = 3072;
  static constexpr int GROUP = NI < 4 ? NI : 4;
  static_assert(NI % GROUP == 0 && (GROUP == 1 || GROUP == 2 || GROUP == 4), "a wave loads 1, 2, 4 or 8 chunks per operand");
  __device__ __forceinline__ void init(int ld, int r0, int wave, int lane, int last_chunks) {
    over = 0;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      int pos = (wave * NI + j) * 64 + lane;
      if (!KS) {
        int row = pos / CH, kc = (pos % CH) ^ rswz(row);
        voff[j] = ((r0 + row) * ld + kc * 8) * 2;
        if (MASKED && kc >= last_chunks) over |= 1u << j;
      } else {
        int krow = pos / (R / 8), c = (pos % (R / 8)) ^ kswz(krow);
        voff[j] = (krow * ld + r0 + c * 8) * 2;
      }
      voff[j] += BIAS - (j % GROUP) * 1024;
      if (MASKED) vfull[j] = voff[j];
    }
  }
  // the next k-tile to be requested is (or is not) the short one at the end of a segment
  __device__ __forceinline__ void set_short(bool is_short) {
    if constexpr (MASKED) {
#pragma unroll
      for (int j = 0; j < NI; ++j) voff[j] = is_short && ((over >> j) & 1) ? (int)0x80000000 : vfull[j];
    }
  }
  // Request one k-step's slab.  rs: buffer resource whose base is the slab's first element minus
  // BIAS bytes and whose num_records is the number of valid bytes from the slab's first element
  // plus BIAS (BIAS itself = nothing to read); LDS_OFF: byte offset of the tile in LDS (ring slot
  // and operand; a constant); wave_off = wave * NI * 1024.  Issued from inline assembly on
  // purpose: through the compiler builtin every LDS read that follows waits for ALL outstanding
  // loads (the compiler cannot tell the ring slots apart), which would undo the multi-stage
  // pipeline.  The kernel keeps its own count instead (s_waitcnt vmcnt(n) before the barrier).
  static constexpr int NGROUPS = NI / GROUP;
  // one group (G0 = its first chunk) of the k-tile's requests
  template <int LDS_OFF, int G0>
  __device__ __forceinline__ void load_group(int4v rs, int wave_off) const {
    // Two hazards the hardware does not interlock and the compiler cannot see inside an asm
    // block (CDNA3 ISA guide, manually inserted wait states): a scalar write of the resource
    // registers needs 5 wait states before a vector-memory instruction reads them (the compiler
    // assembles the 4-register tuple right before the block: s_nop 4), and a scalar write of M0
    // needs 1 before the LDS-direct load that uses it (s_nop 0).  One block per group, so that
    // nothing the compiler emits can come between the M0 write and its loads.
    if constexpr (GROUP == 4) {
      asm volatile(
          "s_nop 4\n\ts_add_u32 m0, %0, %1\n\ts_nop 0\n\t"
          "buffer_load_dwordx4 %2, %6, 0 offen lds\n\t"
          "buffer_load_dwordx4 %3, %6, 0 offen offset:1024 lds\n\t"
          "buffer_load_dwordx4 %4, %6, 0 offen offset:2048 lds\n\t"
          "buffer_load_dwordx4 %5, %6, 0 offen offset:3072 lds"
          :
          : "s"(wave_off), "i"(LDS_OFF + G0 * 1024), "v"(voff[G0]), "v"(voff[G0 + 1]), "v"(voff[G0 + 2]),
            "v"(voff[G0 + 3]), "s"(rs)
          : "memory", "m0", "scc");
    } else if constexpr (GROUP == 1) {
      asm volatile(
          "s_nop 4\n\ts_add_u32 m0, %0, %1\n\ts_nop 0\n\t"
          "buffer_load_dwordx4 %2, %3, 0 offen lds"
          :
          : "s"(wave_off), "i"(LDS_OFF + G0 * 1024), "v"(voff[G0]), "s"(rs)
          : "memory", "m0", "scc");
    } else {
      asm volatile(
          "s_nop 4\n\ts_add_u32 m0, %0, %1\n\ts_nop 0\n\t"
          "buffer_load_dwordx4 %2, %4, 0 offen lds\n\t"
          "buffer_load_dwordx4 %3, %4, 0 offen offset:1024 lds"
          :
          : "s"(wave_off), "i"(LDS_OFF + G0 * 1024), "v"(voff[G0]), "v"(voff[G0 + 1]), "s"(rs)
          : "memory", "m0", "scc");
    }
  }
  template <int LDS_OFF>
  __device__ __forceinline__ void load(int4v rs, int wave_off) const {
    static_for<NGROUPS>([&](auto G) { load_group<LDS_OFF, decltype(G)::value * GROUP>(rs, wave_off); });
  }
};

// One k-tile's requests of both operands in one block: the wait states before the first one serve both.
constexpr bool has_load_pair(int na, int nb) { return (na == nb && (na == 1 || na == 2 || na == 4)) || (na == 4 && nb == 2) || (na == 2 && nb == 4); }
template <int A_OFF, int B_OFF, typename TA, typename TB>
__device__ __forceinline__ void load_pair(const TA& a, const TB& b, int4v ars, int4v brs, int wave_off_a, int wave_off_b) {
  constexpr int NA = TA::NI, NB = TB::NI;
  if constexpr (NA == 1 && NB == 1) {
    asm volatile(
        "s_nop 4\n\ts_add_u32 m0, %0, %2\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %6, %4, 0 offen lds\n\t"
        "s_add_u32 m0, %1, %3\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %7, %5, 0 offen lds"
        :
        : "s"(wave_off_a), "s"(wave_off_b), "i"(A_OFF), "i"(B_OFF), "s"(ars), "s"(brs), "v"(a.voff[0]), "v"(b.voff[0])
        : "memory", "m0", "scc");
  } else if constexpr (NA == 2 && NB == 2) {
    asm volatile(
        "s_nop 4\n\ts_add_u32 m0, %0, %2\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %6, %4, 0 offen lds\n\t"
        "buffer_load_dwordx4 %7, %4, 0 offen offset:1024 lds\n\t"
        "s_add_u32 m0, %1, %3\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %8, %5, 0 offen lds\n\t"
        "buffer_load_dwordx4 %9, %5, 0 offen offset:1024 lds"
        :
        : "s"(wave_off_a), "s"(wave_off_b), "i"(A_OFF), "i"(B_OFF), "s"(ars), "s"(brs), "v"(a.voff[0]), "v"(a.voff[1]),
          "v"(b.voff[0]), "v"(b.voff[1])
        : "memory", "m0", "scc");
  } else if constexpr (NA == 4 && NB == 4) {
    asm volatile(
        "s_nop 4\n\ts_add_u32 m0, %0, %2\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %6, %4, 0 offen lds\n\t"
        "buffer_load_dwordx4 %7, %4, 0 offen offset:1024 lds\n\t"
        "buffer_load_dwordx4 %8, %4, 0 offen offset:2048 lds\n\t"
        "buffer_load_dwordx4 %9, %4, 0 offen offset:3072 lds\n\t"
        "s_add_u32 m0, %1, %3\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %10, %5, 0 offen lds\n\t"
        "buffer_load_dwordx4 %11, %5, 0 offen offset:1024 lds\n\t"
        "buffer_load_dwordx4 %12, %5, 0 offen offset:2048 lds\n\t"
        "buffer_load_dwordx4 %13, %5, 0 offen offset:3072 lds"
        :
        : "s"(wave_off_a), "s"(wave_off_b), "i"(A_OFF), "i"(B_OFF), "s"(ars), "s"(brs), "v"(a.voff[0]), "v"(a.voff[1]),
          "v"(a.voff[2]), "v"(a.voff[3]), "v"(b.voff[0]), "v"(b.voff[1]), "v"(b.voff[2]), "v"(b.voff[3])
        : "memory", "m0", "scc");
  } else if constexpr (NA == 2 && NB == 4) {
    asm volatile(
        "s_nop 4\n\ts_add_u32 m0, %0, %2\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %6, %4, 0 offen lds\n\t"
        "buffer_load_dwordx4 %7, %4, 0 offen offset:1024 lds\n\t"
        "s_add_u32 m0, %1, %3\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %8, %5, 0 offen lds\n\t"
        "buffer_load_dwordx4 %9, %5, 0 offen offset:1024 lds\n\t"
        "buffer_load_dwordx4 %10, %5, 0 offen offset:2048 lds\n\t"
        "buffer_load_dwordx4 %11, %5, 0 offen offset:3072 lds"
        :
        : "s"(wave_off_a), "s"(wave_off_b), "i"(A_OFF), "i"(B_OFF), "s"(ars), "s"(brs), "v"(a.voff[0]), "v"(a.voff[1]),
          "v"(b.voff[0]), "v"(b.voff[1]), "v"(b.voff[2]), "v"(b.voff[3])
        : "memory", "m0", "scc");
  } else {
    static_assert(NA == 4 && NB == 2, "see has_load_pair");
    asm volatile(
        "s_nop 4\n\ts_add_u32 m0, %0, %2\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %6, %4, 0 offen lds\n\t"
        "buffer_load_dwordx4 %7, %4, 0 offen offset:1024 lds\n\t"
        "buffer_load_dwordx4 %8, %4, 0 offen offset:2048 lds\n\t"
        "buffer_load_dwordx4 %9, %4, 0 offen offset:3072 lds\n\t"
        "s_add_u32 m0, %1, %3\n\ts_nop 0\n\t"
        "buffer_load_dwordx4 %10, %5, 0 offen lds\n\t"
        "buffer_load_dwordx4 %11, %5, 0 offen offset:1024 lds"
        :
        : "s"(wave_off_a), "s"(wave_off_b), "i"(A_OFF), "i"(B_OFF), "s"(ars), "s"(brs), "v"(a.voff[0]), "v"(a.voff[1]),
          "v"(a.voff[2]), "v"(a.voff[3]), "v"(b.voff[0]), "v"(b.voff[1])
        : "memory", "m0", "scc");
  }
}

// LDS byte addresses of a lane's MFMA fragments, relative to the operand's tile:
// rows w0 + 32*blk + (lane & 31), k = kk*16 + 8*(lane>>5) + 0..7.  Everything that depends
// on blk, kk or the ring slot beyond these few registers is an instruction immediate.
template <int R, bool KS, int NB, int BK>
struct FragAddr {
  static constexpr int KSTEPS = BK / 16;
  unsigned a[KS ? NB : KSTEPS];
  __device__ __forceinline__ void init(int w0, int lane) {
    if (!KS) {
      int r = lane & 31, sw = OperandTile<R, KS, 4, BK>::rswz(r);  // w0 is a multiple of 32: the swizzle sees lane bits only
#pragma unroll
      for (int kk = 0; kk < KSTEPS; ++kk) a[kk] = (unsigned)((w0 + r) * (BK * 2) + (((kk * 2 + (lane >> 5)) ^ sw) << 4));
    } else {
      int i16 = lane & 15, g16 = (lane >> 4) & 1, h = lane >> 5;
      int krow = 8 * h + (i16 >> 2);
      int sw = OperandTile<R, KS, 4, BK>::kswz(i16 >> 2);  // depends on krow & 3 only
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        int col = w0 + 32 * b + 16 * g16 + 4 * (i16 & 3);
        a[b] = (unsigned)((krow * R + (((col >> 3) ^ sw) << 3) + (col & 7)) * 2);
      }
    }
  }
  // OFF: byte offset of the operand's tile in LDS (a constant)
  template <int OFF, int BLK, int KK>
  __device__ __forceinline__ bf16x8 get(const unsigned char* smem) const {
    if (!KS) {
      return *(const bf16x8*)(smem + a[KK] + (OFF + BLK * 32 * BK * 2));
    } else {
      const bf16* p = (const bf16*)(smem + a[BLK] + (OFF + KK * 16 * R * 2));
      return join8(lds_read_tr16(p), lds_read_tr16(p + 4 * R));
    }
  }
};

// A lane's 8 or 16 bytes of an output.
// Through: written through to memory.  What a launch leaves dirty in the eight L2s (32 MB) is written back when it ends,
// with nothing beside it; the large tiles, whose launches write that much and more, send it on while other tiles still
// multiply (6 layers of 1024: 8192 rows 10.66 -> 10.52 ms, with re-computation 28.0 -> 27.7; small launches only lose what
// the next kernel would have found in its L2: one sample 1216 -> 1240 us with all tiles).
// Far: not kept in the caches.  What only the backward task reads again -- GELU', the attention's fp32 output -- is out of
// them by then and takes the place of what the next kernels read (12 layers of 4096 rows 24.93 -> 24.62 ms, 6 of 8192 10.43
// -> 10.38; with smaller tiles too one sample 1214 -> 1219 us, 2 layers of 2048 rows 680 -> 684: what they write is still there).
// Weight gradients summed over several micro-batches likewise: read and written once per group (2 layers of 2048 rows
// 682 -> 676 us, 12 of 4096 24.44 -> 24.31 ms; with non-temporal loads of C too 24.54).
// (Wait states: a store of more than 8 bytes reads its data after issue, and the compiler does not see one in here.)
enum class Store { Plain, Through, Far };
template <Store S, typename V>
__device__ __forceinline__ void store_c(void* p, V v) {
  typedef float fv __attribute__((__vector_size__(sizeof(V))));
  const fv x = __builtin_bit_cast(fv, v);
  if constexpr (S == Store::Plain) *(fv*)p = x;
  else if constexpr (S == Store::Far) __builtin_nontemporal_store(x, (fv*)p);
  else if constexpr (sizeof(V) == 8) asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(p), "v"(x) : "memory");
  else asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(x) : "memory");
}

// sum over each group of 8 consecutive lanes, in every lane of the group, as a fixed tree: lane pairs, pairs of
// pairs (both inside a quad), then the two quads (the mirror image within the half row) -- cross-lane operands of
// the adds themselves, no trip through LDS
__device__ __forceinline__ float sum8(float v) {
  auto dpp = [](float x, auto CTRL) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(CTRL)::value, 0xF, 0xF, true));
  };
  v += dpp(v, std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
  v += dpp(v, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  v += dpp(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
  return v;
}

template <int BM, int BN, int WGM, int WGN, int NS, bool AKS, bool BKS, int BK, bool KT = false, bool SEG = false>
struct GemmTile {
  static constexpr int NW = WGM * WGN, NT = 64 * NW;
  static constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NI = WN / 32;
  typedef OperandTile<BM, AKS, NW, BK, KT> TA;
  typedef OperandTile<BN, BKS, NW, BK, KT> TB;
  static constexpr int STAGE_ELEMS = TA::LDS_ELEMS + TB::LDS_ELEMS;
  static constexpr int EPI_LD = WN + 4;  // fp32 staging row
  static constexpr size_t MAIN_BYTES = NS * (size_t)STAGE_ELEMS * sizeof(bf16);
  static constexpr int LOADS_PER_TILE = TA::NI + TB::NI;  // per wave
  static constexpr size_t EPI_BYTES = (size_t)NW * 32 * EPI_LD * sizeof(float);
  static constexpr size_t LDS_BYTES = MAIN_BYTES > EPI_BYTES ? MAIN_BYTES : EPI_BYTES;
  // Fragments are read from LDS a whole k-tile ahead of their MFMAs (two sets of them) instead of one k-step: where a
  // wave's k-step is one or two MFMAs (32 or 64 clocks) and no other wave shares its SIMD, an LDS round trip per k-step
  // is what such a loop takes.
  static constexpr bool AHEAD = NW <= 4 && MI * NI <= 2 && NS % 2 == 0;
  // waves per SIMD the registers must allow: two workgroups where LDS has room for them
  static constexpr bool TWO = LDS_BYTES <= 80 * 1024;
  static constexpr int MIN_WAVES = !SEG && NW == 8 && TWO ? 4 : (SEG || (NW == 4 && TWO) ? 2 : 1);
};

// CS: the variant that can also sum B over k (EPI_BSUM); KT: the variant for K segments that are no multiple of 64
// when an operand is k-contiguous (see OperandTile); SEG: an accumulating product over several K segments, each one's
// sum added to C on its own, in order (EPI_SEGACC): a second set of accumulators holds C and takes the sums of the
// segments as they are complete, so C is read and written once whatever their number; PACK: the k-tiles of several
// segments follow each other without a gap (see packs)
template <int BM, int BN, int WGM, int WGN, int NS, bool AKS, bool BKS, int BK, bool CS, bool KT = false, bool SEG = false, bool PACK = false>
__device__ __forceinline__ void gemm_mfma_tile(const GemmArgs& g, int tiles_m, int tiles_n, const int bid, const int z) {
  typedef GemmTile<BM, BN, WGM, WGN, NS, AKS, BKS, BK, KT, SEG> CFG;
  typedef typename CFG::TA TA;
  typedef typename CFG::TB TB;
  constexpr int MI = CFG::MI, NI = CFG::NI;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave / WGN) * CFG::WM, wn0 = (wave % WGN) * CFG::WN;

  int tm, tn;
  tile_of(bid, tiles_m, tiles_n, BM, BN, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  // (the small tiles: every argument the prologue and the first requests need in one go of scalar loads, not a round trip
  // per branch that uses some.  Not the 128x64 tile in eight waves, 80 registers a lane, 102 with it: 1400 x 1024 x 4096 21.2
  // us, 22.4 with it, gradient 20.3 and 21.7, with cold weights 31.9 and 32.4)
  constexpr bool EARLY = CFG::NW <= 4 && MI * (CFG::WN / 8) <= 8;
  if constexpr (EARLY)
    asm volatile("" ::"s"(g.A), "s"(g.B), "s"(g.C), "s"(g.bias), "s"(g.aux), "s"(g.M), "s"(g.N), "s"(g.K), "s"(g.lda), "s"(g.ldb),
                 "s"(g.ldc), "s"(g.ldaux), "s"(g.kseg_len), "s"(g.segA), "s"(g.segB), "s"(g.ln_stats), "s"(g.ln_gamma),
                 "s"(g.ln_beta), "s"(g.k_valid), "s"(g.m_valid), "s"(g.n_valid), "s"(g.epi));

  const bf16 *Ab = (const bf16*)g.A + z * g.sA, *Bb = (const bf16*)g.B + z * g.sB;
  void* const Cb = g.C;
  // (whole turns of the ring per segment, PACK: in all; the k-tiles beyond the end read nothing)
  const int seg_tiles = (g.kseg_len + BK - 1) / BK;
  const int turns = (seg_tiles + NS - 1) / NS;   // of the ring, per segment
  const int k_rows = g.K > g.kseg_len ? g.kseg_len : g.k_valid;   // rows of one segment of a k-strided operand
  // bytes of one segment of each operand that may be read (beyond: zero)
  const long a_ext =
      AKS ? ((long)(k_rows - 1) * g.lda + g.m_valid) * 2 : ((long)(g.m_valid - 1) * g.lda + g.kseg_len) * 2;
  const long b_ext =
      BKS ? ((long)(k_rows - 1) * g.ldb + g.n_valid) * 2 : ((long)(g.n_valid - 1) * g.ldb + g.kseg_len) * 2;

  TA ta;
  TB tb;
  const int last_chunks = (g.kseg_len - (seg_tiles - 1) * BK) / 8;   // 16-byte chunks of a segment's last k-tile
  ta.init(g.lda, m0, wave, lane, last_chunks);
  tb.init(g.ldb, n0, wave, lane, last_chunks);
  ta.set_short(seg_tiles == 1);
  tb.set_short(seg_tiles == 1);
  FragAddr<BM, AKS, MI, BK> fa;
  FragAddr<BN, BKS, NI, BK> fb;
  fa.init(wm0, lane);
  fb.init(wn0, lane);
  int wave_off_a = wave * TA::NI * 1024, wave_off_b = wave * TB::NI * 1024;

  // Global cursors, all in scalar registers: one buffer resource per operand whose base is
  // the first element of the next k-step's slab and whose num_records is what may still be
  // read from there.  A k-step forward is base += step, records -= step; at the end of a
  // K segment the base jumps to the next segment and the records start over.
  // A wave issues an instruction every few clocks, and the small tiles' loop is bound by that: segments are whole turns of
  // the ring, so that only the turn's first slot, which requests the last tile of a turn, looks for a segment's end.
  // (PACK: every slot does.)
  const int a_step = AKS ? BK * g.lda * 2 : BK * 2, b_step = BKS ? BK * g.ldb * 2 : BK * 2;
  const long a_jump = g.segA * 2 - (long)(seg_tiles - 1) * a_step, b_jump = g.segB * 2 - (long)(seg_tiles - 1) * b_step;
  int4v ars, brs;
  auto set_base = [](int4v& rs, uint64_t p) {
    rs[0] = (int)(uint32_t)p;
    rs[1] = (int)(uint32_t)(p >> 32);  // a device address has no bits above 47: stride and swizzle fields stay 0
  };
  auto get_base = [](const int4v& rs) { return ((uint64_t)(uint32_t)rs[1] << 32) | (uint32_t)rs[0]; };
  uint64_t a_seg = (uint64_t)Ab - TA::BIAS, b_seg = (uint64_t)Bb - TB::BIAS;   // of the segment being requested
  set_base(ars, a_seg);
  set_base(brs, b_seg);
  // record counts carry the operand tiles' BIAS (see OperandTile); BIAS alone = nothing readable
  const int a_rec0 = (int)a_ext + TA::BIAS, b_rec0 = (int)b_ext + TB::BIAS;
  ars[2] = a_rec0;
  brs[2] = b_rec0;
  ars[3] = brs[3] = (int)BUF_RSRC_FLAGS;
  // (uniform, and kept in scalar registers: the resources are read by inline assembly)
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    ars[i] = __builtin_amdgcn_readfirstlane(ars[i]);
    brs[i] = __builtin_amdgcn_readfirstlane(brs[i]);
  }
  wave_off_a = __builtin_amdgcn_readfirstlane(wave_off_a);
  wave_off_b = __builtin_amdgcn_readfirstlane(wave_off_b);
  // Branch-free on purpose: with control flow inside the k-loop the accumulators get
  // copied between register files at every merge point.
  // still to be requested (tiles_left: of the segment, PACK: in all)
  int turns_left = turns, segs_left = g.K / g.kseg_len, seg_left = seg_tiles, tiles_left = PACK ? segs_left * seg_tiles : seg_tiles;
  auto advance = [&](auto S) __attribute__((always_inline)) {
    --tiles_left;
    if constexpr (PACK) {
      const bool cross = --seg_left == 0, more = tiles_left > 0;
      set_base(ars, get_base(ars) + (uint64_t)(cross ? a_jump : (long)a_step));
      set_base(brs, get_base(brs) + (uint64_t)(cross ? b_jump : (long)b_step));
      ars[2] = more ? (cross ? a_rec0 : max(ars[2] - a_step, (int)TA::BIAS)) : (int)TA::BIAS;
      brs[2] = more ? (cross ? b_rec0 : max(brs[2] - b_step, (int)TB::BIAS)) : (int)TB::BIAS;
      seg_left = cross ? seg_tiles : seg_left;
      ta.set_short(seg_left == 1);
      tb.set_short(seg_left == 1);
      return;
    }
    set_base(ars, get_base(ars) + (uint32_t)a_step);
    set_base(brs, get_base(brs) + (uint32_t)b_step);
    int ar = max(ars[2] - a_step, (int)TA::BIAS), br = max(brs[2] - b_step, (int)TB::BIAS);
    if constexpr (decltype(S)::value == 0) {   // the request before was the last of its turn
      const bool cross = --turns_left == 0;
      segs_left -= cross;
      a_seg += cross ? (uint64_t)(g.segA * 2) : 0;
      b_seg += cross ? (uint64_t)(g.segB * 2) : 0;
      set_base(ars, cross ? a_seg : get_base(ars));
      set_base(brs, cross ? b_seg : get_base(brs));
      ar = cross ? a_rec0 : ar;
      br = cross ? b_rec0 : br;
      tiles_left = cross ? (segs_left > 0 ? seg_tiles : 0) : tiles_left;
      turns_left = cross ? turns : turns_left;
    }
    // past a segment's last k-tile the cursor reads nothing: such a request fills its slot with zeros
    ars[2] = tiles_left > 0 ? ar : (int)TA::BIAS;
    brs[2] = tiles_left > 0 ? br : (int)TB::BIAS;
    ta.set_short(tiles_left == 1);
    tb.set_short(tiles_left == 1);
  };
  constexpr bool PAIR = has_load_pair(TA::NI, TB::NI);   // one block requests a tile's part of both operands
  // request the next k-tile into ring slot S
  auto issue_loads = [&](auto S) {
    constexpr int off = decltype(S)::value * CFG::STAGE_ELEMS * 2;
    if constexpr (PAIR) {
      load_pair<off, off + TA::LDS_BYTES>(ta, tb, ars, brs, wave_off_a, wave_off_b);
    } else {
      ta.template load<off>(ars, wave_off_a);
      tb.template load<off + TA::LDS_BYTES>(brs, wave_off_b);
    }
    advance(std::integral_constant<int, NS == 1 ? 0 : (decltype(S)::value + 1) % NS>{});
  };

  // The epilogue's reads.  A wave's vector-memory requests complete in the order they were issued, stores among them:
  // waiting for a value requested AFTER a store waits for the store's acknowledgement as well.  So nothing is requested
  // between two blocks' stores that is not needed until the block after: the bias (the same four columns for every row
  // a lane stores) is read once, and the second operand (residual, gate) or the fp32 C of an accumulating product is
  // requested one unit (16 or 32 rows) ahead -- the first one's before the workgroup's last barrier and the staging of
  // the accumulators through LDS -- or all of it there where the registers allow (PRE: the tiles with at most 64 rows
  // per wave); or, in the small tiles, before the first k-tile (EARLY): a launch of those is mostly memory latencies in
  // a row, and this takes one of them off.
  const long zc = z * g.sC, zbias = z * g.sBias;
  constexpr int C4 = CFG::WN / 4;             // float4 per staged row
  constexpr int NIT = 32 * C4 / 64;           // float4 per lane per 32-row block
  static_assert(64 % C4 == 0, "a lane stores the same columns of every row");
  constexpr int HB = MI > 2 ? (NIT > 4 ? 4 : NIT) : (NIT > 8 ? 8 : NIT);   // processed HB at a time
  constexpr Store THROUGH = BM == 256 ? Store::Through : Store::Plain, FAR = BM == 256 ? Store::Far : Store::Plain;
  constexpr bool PRE = !CS && !SEG && MI * NIT <= 16;   // (the column-sum variant serves accumulating products only)
  const int epi = g.epi;
  const int lane_col = n0 + wn0 + lane % C4 * 4;   // the lane's four columns
  const bool interior = m0 + BM <= g.M && n0 + BN <= g.N;
  // What a product's epilogue reads, as a constant: flags tested per request have the loads wait for each other where
  // the branches meet (gate of 8192 x 4096 x 1024: 108 us, 89 with the whole operand requested in one go).
  //   AUXH: a bf16 second operand, all of it ahead; AUXF: an fp32 one; AUXL: one whose LayerNorm is added (EPI_AUXLN);
  //   ACCF: the fp32 C of an accumulating product;
  //   ANY: nothing ahead (no operand, or a combination that no product of the stage has, read in place)
  enum { AUXH, AUXF, AUXL, ACCF, ANY };
  const bool has_aux = (epi & (EPI_ADD | EPI_MUL | EPI_ROWDOT)) != 0, has_acc = (epi & EPI_ACC32) != 0;
  auto with_mode = [&](auto&& f) __attribute__((always_inline)) {
    constexpr bool TT = AKS && BKS;   // the weight-gradient layout: the only one that accumulates
    if constexpr (SEG) {
      // (C is in the second set of accumulators)
    } else if constexpr (TT) {
      if (has_acc && !has_aux) return f(std::integral_constant<int, ACCF>{});
    } else {
      if (has_aux && !has_acc) {
        if (epi & EPI_AUXLN) return f(std::integral_constant<int, AUXL>{});
        if (epi & EPI_AUX32) return f(std::integral_constant<int, AUXF>{});
        if (!(epi & EPI_ROWDOT)) return f(std::integral_constant<int, AUXH>{});
      }
    }
    return f(std::integral_constant<int, ANY>{});
  };
  // (native vectors: arrays of the runtime's float4, a struct around a union, stay in scratch memory)
  typedef float f32x2 __attribute__((__vector_size__(2 * sizeof(float))));
  constexpr int UNITS = MI * (NIT / HB);
  f32x4 pre[PRE ? UNITS : 2][HB];    // fp32 operands: whole (PRE), or the unit in use and the one after
  f32x2 preh[UNITS][HB];             // a bf16 operand
  // AUXL: mean and rstd of the wave's row 64 i + lane; in the small tiles, of each piece's row (no exchange at the end)
  f32x2 rstat[EARLY ? UNITS * HB : (MI + 1) / 2];
  f32x2 lng{}, lnb{};                // ... gamma and beta of the lane's columns, four bf16 each (converted where they
                                     // are used: a conversion here would wait for the load)
  // Addresses: a lane's piece n of block i is row m0 + wm0 + 32 i + n RS + lane / C4.  All but the last term is the same
  // for the whole wave and stays in scalar registers; a lane keeps one 32-bit offset per matrix (64-bit addresses per
  // piece had the 256x256 tile's accumulators spill).
  constexpr int RS = 64 / C4;
  const unsigned c_off4 = (unsigned)((lane / C4) * g.ldc + lane % C4 * 4) * 4u, a_off4 = (unsigned)((lane / C4) * g.ldaux + lane % C4 * 4) * 4u;
  auto row_of = [&](int i, int n) { return m0 + wm0 + i * 32 + n * RS + lane / C4; };
  auto at = [&](const void* base, int ld, unsigned lane_off, int i, int n, int es) {
    const long u = (zc + (long)(m0 + wm0 + i * 32 + n * RS) * ld + n0 + wn0) * es;
    return (char*)base + u + lane_off;
  };
  // HB pieces of that operand (unit k), as each lane will use them in store_block
  auto request = [&](auto K, auto MODE, auto FULLC) __attribute__((always_inline)) {
    constexpr int k = decltype(K)::value, i = k / (NIT / HB), hb = k % (NIT / HB) * HB, mode = decltype(MODE)::value;
    static_for<HB>([&](auto U) __attribute__((always_inline)) {
      constexpr int u = decltype(U)::value, n = hb + u, slot = PRE ? k : (k & 1);
      const bool in = decltype(FULLC)::value || (row_of(i, n) < g.M && lane_col < g.N);
      if constexpr (mode == AUXH) preh[k][u] = in ? *(const f32x2*)at(g.aux, g.ldaux, a_off4 >> 1, i, n, 2) : f32x2{0.f, 0.f};
      if constexpr (mode == AUXF || mode == AUXL) pre[slot][u] = in ? *(const f32x4*)at(g.aux, g.ldaux, a_off4, i, n, 4) : f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (mode == ACCF) pre[slot][u] = in ? *(const f32x4*)at(Cb, g.ldc, c_off4, i, n, 4) : f32x4{0.f, 0.f, 0.f, 0.f};
    });
  };
  f32x2 bias4{};
  auto request_first = [&](auto MODE, auto FULLC) __attribute__((always_inline)) {
    static_for<PRE || decltype(MODE)::value == AUXH ? UNITS : 1>([&](auto K) __attribute__((always_inline)) { request(K, MODE, FULLC); });
    if constexpr (decltype(MODE)::value == AUXL) {
      if constexpr (EARLY) {
#pragma unroll
        for (int p = 0; p < UNITS * HB; ++p) rstat[p] = *(const f32x2*)(g.ln_stats + 2 * min(row_of(p / NIT, p % NIT), g.M - 1));
      } else {
#pragma unroll
        for (int i = 0; i < (MI + 1) / 2; ++i)
          rstat[i] = *(const f32x2*)(g.ln_stats + 2 * min(m0 + wm0 + 64 * i + (MI > 1 ? lane : lane & 31), g.M - 1));
      }
      if (lane_col < g.N) {
        lng = *(const f32x2*)((const bf16*)g.ln_gamma + lane_col);
        lnb = *(const f32x2*)((const bf16*)g.ln_beta + lane_col);
      }
    }
    if ((epi & EPI_BIAS) && lane_col < g.N) bias4 = *(const f32x2*)((const bf16*)g.bias + zbias + lane_col);
  };
  f32x16 acc[MI][NI], tot[SEG ? MI : 1][SEG ? NI : 1];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  };
  clear();

  // Software pipeline.  Global->LDS: a k-tile is requested NS-1 iterations before it is
  // used, as soon as every wave has left the ring slot it goes to.  LDS->registers: the
  // fragments of k-step kk+1 are requested before the MFMAs of k-step kk are issued (two
  // fragment sets), so the matrix cores wait for an LDS round trip only once per tile.
  struct Frags {
    bf16x8 a[MI], b[NI];
  };
  constexpr int KSTEPS = BK / 16;
  static_assert(KSTEPS % 2 == 0, "the two fragment sets alternate over an even number of k-steps");

  // The loop runs whole turns of the ring: each K segment (PACK: all of K) is padded to a multiple of NS k-tiles
  // with tiles that read nothing (zeros in LDS add nothing), and every iteration requests a tile,
  // so the count of requests in flight is the same in every iteration.
  // vmcnt(N): at most N of this wave's requests still in flight; requests complete in order,
  // so N = (NS - 2) * LOADS_PER_TILE means "tile kt has landed"
  constexpr int INFLIGHT = (NS - 2) * CFG::LOADS_PER_TILE;
  constexpr int C_LOADS = SEG ? MI * NI * 4 : 0;   // SEG: requests for C, in flight behind those for the tiles once
  static_assert(INFLIGHT + C_LOADS < 64, "vmcnt is a 6-bit counter");
  // ... and lgkmcnt(0): this wave's LDS reads of the previous tile must have EXECUTED, not just
  // been issued, before the barrier lets other waves refill that slot (a request that reads
  // nothing delivers its zeros within a few clocks)
  constexpr auto wait_tile = [](int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; };  // expcnt: no wait
  float* const bsum_ptr = CS && z == 0 ? g.bsum : nullptr;
  const bool do_cs = CS && (g.epi & EPI_BSUM) && tm == 0 && wm0 == 0 && bsum_ptr != nullptr;
  float bsum0[NI];   // what the column sums are added to
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    const int col = n0 + wn0 + 32 * j + (lane & 31);
    bsum0[j] = do_cs && lane < 32 && col < g.N ? bsum_ptr[col] : 0.f;
  }
  if constexpr (EARLY) {
    with_mode([&](auto MODE) __attribute__((always_inline)) {
      if (interior) request_first(MODE, std::true_type{});
      else request_first(MODE, std::false_type{});
    });
  }
  static_for<NS - 1>([&](auto T) { issue_loads(T); });
  // The k-steps are rotated by one against the tiles: the MFMAs of a tile's LAST k-step are issued after the
  // barrier that opens the next tile (their fragments were read before it).  Everything else a tile needs --
  // the LDS reads of the next k-step's fragments, the requests for the tile NS - 1 ahead, the cursor arithmetic
  // -- is cut in pieces and placed BETWEEN the MFMAs of a k-step in a fixed order (nothing may be moved across
  // the fences): a wave issues an instruction every few clocks while an MFMA holds the matrix pipe for 32, so
  // in the shadow of each MFMA there is room for a few other instructions and the pipe never waits for them.
  // The very first rotated step multiplies zeros.
  Frags f0, f1;
  static_for<MI>([&](auto I) { f1.a[decltype(I)::value] = bf16x8{}; });
  static_for<NI>([&](auto J) { f1.b[decltype(J)::value] = bf16x8{}; });
  constexpr int GA = TA::NGROUPS, GB = PAIR ? 0 : TB::NGROUPS, EXTRA = GA + GB + 1;  // request groups of A, of B, the cursor step
  constexpr int NFRAG = MI + NI, NM = MI * NI;
  // step J of tile S: the MFMAs of `use`; between them the reads of `fill` (the fragments of k-step J of tile S,
  // in the order the next step's MFMAs need them: a0, b0 .. b_NI-1, a1 ..) and this step's share of the requests
  // for the tile that goes to ring slot SN
  // EPI_BSUM: bsum[n] += sum_k B(n,k) for this tile's columns, by the workgroups of the first tile row (tm == 0)
  // and there by the waves that hold the tile's first rows: each lane adds up the B fragments it holds anyway, two
  // products with one per instruction (exact, fp32 sums), between the MFMAs.  One register per 32 columns: sums
  // taken with MFMAs against a fragment of ones needed sixteen, which two sets of accumulators leave no room for.
  float csum[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) csum[j] = 0.f;
  const bf16x2 one2 = {(bf16)1.0f, (bf16)1.0f};
  auto add_cols = [&](float& t, bf16x8 b) {
    t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 0, 1), one2, t, false);
    t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 2, 3), one2, t, false);
    t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 4, 5), one2, t, false);
    t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 6, 7), one2, t, false);
  };
  auto step = [&](const Frags& use, Frags& fill, auto S, auto SN, auto J, auto WCS) {
    constexpr int off = decltype(S)::value * CFG::STAGE_ELEMS * 2, offn = decltype(SN)::value * CFG::STAGE_ELEMS * 2;
    constexpr int j = decltype(J)::value;
    constexpr int e0 = j * EXTRA / KSTEPS, e1 = (j + 1) * EXTRA / KSTEPS, P = NFRAG + (e1 - e0);
    static_for<NM>([&](auto Q) {
      constexpr int q = decltype(Q)::value, mi = q / NI, ni = q % NI;
      acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(use.b[ni], use.a[mi], acc[mi][ni], 0, 0, 0);
      if constexpr (decltype(WCS)::value && mi == 0) add_cols(csum[ni], use.b[ni]);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int p0 = q * P / NM, p1 = (q + 1) * P / NM;
      static_for<p1 - p0>([&](auto D) {
        constexpr int p = p0 + decltype(D)::value;
        if constexpr (p == 0) {
          fill.a[0] = fa.template get<off, 0, j>(smem);
        } else if constexpr (p <= NI) {
          fill.b[p - 1] = fb.template get<off + TA::LDS_BYTES, p - 1, j>(smem);
        } else if constexpr (p < NFRAG) {
          fill.a[p - NI] = fa.template get<off, p - NI, j>(smem);
        } else {
          constexpr int e = e0 + (p - NFRAG);
          if constexpr (PAIR && e == 0) load_pair<offn, offn + TA::LDS_BYTES>(ta, tb, ars, brs, wave_off_a, wave_off_b);
          else if constexpr (e < GA) ta.template load_group<offn, e * TA::GROUP>(ars, wave_off_a);
          else if constexpr (e < GA + GB) tb.template load_group<offn + TA::LDS_BYTES, (e - GA) * TB::GROUP>(brs, wave_off_b);
          else advance(S);
        }
      });
      if constexpr (p1 > p0) __builtin_amdgcn_sched_barrier(0);
    });
  };
  // AHEAD: a whole tile at once.  The MFMAs of tile t - 1, whose fragments were read during the tile before, and between
  // them -- the reads first, they are what the next barrier waits for -- the reads of tile t's fragments and the requests.
  constexpr bool AHEAD = CFG::AHEAD;
  Frags fs[AHEAD ? 2 : 1][AHEAD ? KSTEPS : 1];
  auto clear_frags = [&](auto& f) __attribute__((always_inline)) {
    static_for<MI>([&](auto I) { f.a[decltype(I)::value] = bf16x8{}; });
    static_for<NI>([&](auto J) { f.b[decltype(J)::value] = bf16x8{}; });
  };
  auto tile_step = [&](auto& use, auto& fill, auto S, auto SN, auto WCS) __attribute__((always_inline)) {
    constexpr int off = decltype(S)::value * CFG::STAGE_ELEMS * 2, offn = decltype(SN)::value * CFG::STAGE_ELEMS * 2;
    constexpr int NMT = NM * KSTEPS, READS = NFRAG * KSTEPS, P = READS + EXTRA, RATE = (P + NMT - 2) / (NMT - 1);
    static_for<NMT>([&](auto Q) {
      constexpr int q = decltype(Q)::value, kk = q / NM, mi = q % NM / NI, ni = q % NI;
      acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(use[kk].b[ni], use[kk].a[mi], acc[mi][ni], 0, 0, 0);
      if constexpr (decltype(WCS)::value && mi == 0) add_cols(csum[ni], use[kk].b[ni]);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int p0 = q * RATE < P ? q * RATE : P, p1 = (q + 1) * RATE < P ? (q + 1) * RATE : P;
      static_for<p1 - p0>([&](auto D) {
        constexpr int p = p0 + decltype(D)::value;
        if constexpr (p < READS) {
          constexpr int k = p / NFRAG, f = p % NFRAG;   // in the order the MFMAs need them
          if constexpr (f == 0) fill[k].a[0] = fa.template get<off, 0, k>(smem);
          else if constexpr (f <= NI) fill[k].b[f - 1] = fb.template get<off + TA::LDS_BYTES, f - 1, k>(smem);
          else fill[k].a[f - NI] = fa.template get<off, f - NI, k>(smem);
        } else {
          constexpr int e = p - READS;
          if constexpr (PAIR && e == 0) load_pair<offn, offn + TA::LDS_BYTES>(ta, tb, ars, brs, wave_off_a, wave_off_b);
          else if constexpr (e < GA) ta.template load_group<offn, e * TA::GROUP>(ars, wave_off_a);
          else if constexpr (e < GA + GB) tb.template load_group<offn + TA::LDS_BYTES, (e - GA) * TB::GROUP>(brs, wave_off_b);
          else advance(S);
        }
      });
      if constexpr (p1 > p0) __builtin_amdgcn_sched_barrier(0);
    });
  };
  if constexpr (AHEAD) static_for<KSTEPS>([&](auto K) { clear_frags(fs[1][decltype(K)::value]); });
  // one turn of the ring; EXTRA_IN: requests in flight besides those for tiles, issued right before it
  auto turn = [&](auto WCS, auto EXTRA_IN) __attribute__((always_inline)) {
    static_for<NS>([&](auto S) {
      typedef std::integral_constant<int, (decltype(S)::value + NS - 1) % NS> SN;
      constexpr int inflight = INFLIGHT + (decltype(S)::value < NS - 1 ? decltype(EXTRA_IN)::value : 0);
      __builtin_amdgcn_sched_barrier(0);  // no LDS read of the previous tile may sink below the barrier
      __builtin_amdgcn_s_waitcnt(wait_tile(inflight));
      __builtin_amdgcn_s_barrier();  // every wave's part of this tile is in LDS; the previous tile's slot is free
      asm volatile("" ::: "memory");  // ... and no LDS read of this tile may be hoisted above it
      if constexpr (AHEAD) tile_step(fs[(decltype(S)::value + 1) & 1], fs[decltype(S)::value & 1], S, SN{}, WCS);
      else static_for<KSTEPS / 2>([&](auto H) {
        constexpr int kk = 2 * decltype(H)::value;
        step(f1, f0, S, SN{}, std::integral_constant<int, kk>{}, WCS);      // MFMAs of k-step kk - 1 (the previous tile's last when kk == 0)
        step(f0, f1, S, SN{}, std::integral_constant<int, kk + 1>{}, WCS);
      });
    });
  };
  // what the last tile left: its last k-step (AHEAD: all of it)
  auto last_step = [&](auto WCS) __attribute__((always_inline)) {
    static_for<AHEAD ? KSTEPS : 1>([&](auto K) {
      const Frags& f = AHEAD ? fs[AHEAD ? (NS - 1) & 1 : 0][decltype(K)::value] : f1;
      static_for<NM>([&](auto Q) {
        constexpr int q = decltype(Q)::value, mi = q / NI, ni = q % NI;
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[ni], f.a[mi], acc[mi][ni], 0, 0, 0);
        if constexpr (decltype(WCS)::value && mi == 0) add_cols(csum[ni], f.b[ni]);
      });
    });
  };
  constexpr std::integral_constant<int, 0> none{};
  // SEG: C, straight into the accumulators' layout, requested before the last turn of the first segment.  A wave's
  // requests complete in order, so the first tile requested after them waits for them too: NS - 1 tiles later.  Every
  // lane issues every request (the waits count them): what lies outside the matrix reads some element inside it.
  auto request_c = [&]() __attribute__((always_inline)) {
    if constexpr (SEG) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const float* row = (const float*)Cb + zc + (long)min(m0 + wm0 + 32 * i + (lane & 31), g.M - 1) * g.ldc;
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 c = *(const f32x4*)(row + min(n0 + wn0 + 32 * j + 8 * q + 4 * (lane >> 5), g.N - 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[i][j][4 * q + e] = c[e];
          }
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // a segment's sums are complete: add them up, start the next one (its first rotated step multiplies zeros again)
  auto end_segment = [&](auto WCS) __attribute__((always_inline)) {
    last_step(WCS);
    if constexpr (SEG) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) tot[i][j] += acc[i][j];
      clear();
      if constexpr (AHEAD) static_for<KSTEPS>([&](auto K) { clear_frags(fs[1][decltype(K)::value]); });
      else clear_frags(f1);
    }
    if constexpr (decltype(WCS)::value) {
      // the two half waves hold the sums over different k
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        bsum0[j] += csum[j] + __shfl_xor(csum[j], 32, 64);
        csum[j] = 0.f;
      }
    }
  };
  auto main_loop = [&](auto WCS) __attribute__((always_inline)) {
    if constexpr (SEG) {
      for (int t = 1; t < turns; ++t) turn(WCS, none);
      request_c();
      turn(WCS, std::integral_constant<int, C_LOADS>{});
      end_segment(WCS);
      for (int s = g.K / g.kseg_len; s > 1; --s) {
        for (int t = 0; t < turns; ++t) turn(WCS, none);
        end_segment(WCS);
      }
    } else {
      for (int t = PACK ? (g.K / g.kseg_len * seg_tiles + NS - 1) / NS : g.K / g.kseg_len * turns; t > 0; --t) turn(WCS, none);
      end_segment(WCS);
    }
  };
  // (two copies of the loop under one uniform branch, none inside it)
  if constexpr (CS) {
    if (do_cs) main_loop(std::true_type{});
    else main_loop(std::false_type{});
  } else {
    main_loop(std::false_type{});
  }
  if constexpr (CS) {
    if (do_cs) {   // (one workgroup per column range adds to bsum: no atomic)
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int col = n0 + wn0 + 32 * j + (lane & 31);
        if (lane < 32 && col < g.N) bsum_ptr[col] = bsum0[j];
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // the tail requests (they read nothing) must be done before LDS is reused
  // epilogue: per wave, 32 output rows at a time through an fp32 LDS staging tile that
  // turns "a lane owns 4 columns of one row" into row-contiguous stores.
  // acc[i][j][v]: row = wm0 + 32 i + (lane & 31), col = wn0 + 32 j + 8 (v>>2) + 4 (lane>>5) + (v&3)
  // All LDS reads of a half block are issued before the first use,
  // so their latencies overlap instead of adding up.
  float* stg = (float*)smem + wave * 32 * CFG::EPI_LD;
  // one 32-row block; the block index is a compile-time constant so that the
  // accumulators are always addressed statically (they must stay in registers)
  auto store_block = [&](auto I, auto FULLC, auto MODE) __attribute__((always_inline)) {
    constexpr int i = decltype(I)::value, mode = decltype(MODE)::value;
    // FULL: the whole tile lies inside the matrix, no element needs a bounds test
    constexpr bool FULL = decltype(FULLC)::value;
    auto stage = [&](auto& acc, float* stg) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float4 v4 = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
          *(float4*)(stg + (lane & 31) * CFG::EPI_LD + j * 32 + 8 * q + 4 * (lane >> 5)) = v4;
        }
    };
    if constexpr (SEG) stage(tot, stg);
    else stage(acc, stg);
    // the staging tile is private to the wave and a wave's LDS instructions execute in
    // order: no workgroup barrier is needed (one would also wait for the stores below)
    __builtin_amdgcn_wave_barrier();
    static_for<NIT / HB>([&](auto Hc) __attribute__((always_inline)) {
      constexpr int hb = decltype(Hc)::value * HB, k = i * (NIT / HB) + decltype(Hc)::value;
      if constexpr (!PRE && mode != AUXH && k + 1 < UNITS) request(std::integral_constant<int, k + 1>{}, MODE, FULLC);   // ahead of this unit's stores
      f32x4 (&in)[HB] = pre[PRE ? k : (k & 1)];
      float4 t[HB];
      bool ok[HB];
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        const int r = ((hb + u) * 64 + lane) / C4;
        ok[u] = FULL || (row_of(i, hb + u) < g.M && lane_col < g.N);
        t[u] = *(const float4*)(stg + r * CFG::EPI_LD + lane % C4 * 4);
      }
      if (epi & EPI_BIAS) {
        const bf16x4 bv = __builtin_bit_cast(bf16x4, bias4);
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          t[u].x += (float)bv[0]; t[u].y += (float)bv[1]; t[u].z += (float)bv[2]; t[u].w += (float)bv[3];
        }
      }
      if (mode == AUXH || mode == AUXF || mode == AUXL || (mode == ANY && has_aux)) {
        float4 xv[HB];
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          f32x4 x{0.f, 0.f, 0.f, 0.f};
          f32x2 h{0.f, 0.f};
          bool half = mode == AUXH;
          if constexpr (mode == AUXH) h = preh[k][u];
          if constexpr (mode == AUXF) x = in[u];
          if constexpr (mode == AUXL) {
            const bf16x4 gv = __builtin_bit_cast(bf16x4, lng), bv = __builtin_bit_cast(bf16x4, lnb);
            const int r = (i & 1) * 32 + (hb + u) * RS + lane / C4;
            const f32x2 st = rstat[EARLY ? i * NIT + hb + u : i / 2];
            const float mean = EARLY ? st[0] : __shfl(st[0], r, 64), rstd = EARLY ? st[1] : __shfl(st[1], r, 64);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = (in[u][e] - mean) * rstd * (float)gv[e] + (float)bv[e];
          }
          if constexpr (mode == ANY) {
            half = !(epi & EPI_AUX32);
            if (half) h = ok[u] ? *(const f32x2*)at(g.aux, g.ldaux, a_off4 >> 1, i, hb + u, 2) : h;
            else x = ok[u] ? *(const f32x4*)at(g.aux, g.ldaux, a_off4, i, hb + u, 4) : x;
          }
          if (half) {
            const bf16x4 b4 = __builtin_bit_cast(bf16x4, h);
            xv[u] = make_float4((float)b4[0], (float)b4[1], (float)b4[2], (float)b4[3]);
          } else {
            xv[u] = make_float4(x[0], x[1], x[2], x[3]);
          }
        }
        if (mode != AUXH && mode != AUXL && (epi & EPI_ROWDOT)) {
          // a row's 32 columns of a block sit in 8 consecutive lanes (4 columns each): products of the
          // outputs as they are stored, summed over the lane's four, then over the eight lanes in a fixed tree
#pragma unroll
          for (int u = 0; u < HB; ++u) {
            float part = (float)(bf16)t[u].x * xv[u].x + (float)(bf16)t[u].y * xv[u].y +
                         (float)(bf16)t[u].z * xv[u].z + (float)(bf16)t[u].w * xv[u].w;
            part = ok[u] ? part : 0.f;
            part = sum8(part);
            if (ok[u] && (lane & 7) == 0) g.rowdot[(long)(lane_col >> 5) * g.M + row_of(i, hb + u)] = part;
          }
        } else {
#pragma unroll
          for (int u = 0; u < HB; ++u) {
            if (epi & EPI_ADD) {
              t[u].x += xv[u].x; t[u].y += xv[u].y; t[u].z += xv[u].z; t[u].w += xv[u].w;
            } else {
              t[u].x *= xv[u].x; t[u].y *= xv[u].y; t[u].z *= xv[u].z; t[u].w *= xv[u].w;
            }
          }
        }
      }
      if (SEG || (epi & EPI_OUT32)) {   // (SEG: C is in the sum already)
#pragma unroll
        for (int u = 0; u < HB; ++u)
          if (ok[u]) store_c<SEG ? Store::Far : THROUGH>(at(Cb, g.ldc, c_off4, i, hb + u, 4), f32x4{t[u].x, t[u].y, t[u].z, t[u].w});
      } else if (mode == ACCF || (mode == ANY && has_acc)) {
        float4 cv[HB];
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          if constexpr (mode == ACCF) cv[u] = make_float4(in[u][0], in[u][1], in[u][2], in[u][3]);
          else cv[u] = ok[u] ? *(const float4*)at(Cb, g.ldc, c_off4, i, hb + u, 4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          cv[u].x += t[u].x; cv[u].y += t[u].y; cv[u].z += t[u].z; cv[u].w += t[u].w;
          if (ok[u]) *(float4*)at(Cb, g.ldc, c_off4, i, hb + u, 4) = cv[u];
        }
      } else if (epi & EPI_GELU) {
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          float tv[4] = {t[u].x, t[u].y, t[u].z, t[u].w};
          bf16x4 gv, gp;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float a, b;
            gelu_both(tv[e], a, b);
            gv[e] = (bf16)a;
            gp[e] = (bf16)b;
          }
          if (ok[u]) {
            store_c<THROUGH>(at(Cb, g.ldc, c_off4 >> 1, i, hb + u, 2), gv);
            store_c<FAR>(at(g.C2, g.ldc, c_off4 >> 1, i, hb + u, 2), gp);
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < HB; ++u) {
          bf16x4 ov;
          ov[0] = (bf16)t[u].x; ov[1] = (bf16)t[u].y; ov[2] = (bf16)t[u].z; ov[3] = (bf16)t[u].w;
          if (ok[u]) store_c<THROUGH>(at(Cb, g.ldc, c_off4 >> 1, i, hb + u, 2), ov);
        }
      }
      __builtin_amdgcn_sched_barrier(0);   // (no unit's reads may be hoisted over another's stores: registers)
    });
    __builtin_amdgcn_wave_barrier();
  };
  auto finish = [&](auto MODE, auto FULLC) __attribute__((always_inline)) {
    if constexpr (!EARLY) request_first(MODE, FULLC);
    // every wave has read its last fragments (lgkmcnt(0)): LDS can be reused after the barrier.  The raw barrier on
    // purpose: __syncthreads() would also wait for the requests just issued.
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<MI>([&](auto I) __attribute__((always_inline)) { store_block(I, FULLC, MODE); });
  };
  // interior tiles (nearly all of them) take the path without per-element bounds tests
  with_mode([&](auto MODE) __attribute__((always_inline)) {
    if (interior) finish(MODE, std::true_type{});
    else finish(MODE, std::false_type{});
  });
  static_assert(MI <= 4, "at most four 32-row blocks per wave");
}

template <int BM, int BN, int WGM, int WGN, int NS, bool AKS, bool BKS, int BK, bool CS, bool KT = false, bool SEG = false, bool PACK = false>
__global__ __launch_bounds__(64 * WGM * WGN, (GemmTile<BM, BN, WGM, WGN, NS, AKS, BKS, BK, KT, SEG>::MIN_WAVES)) void gemm_mfma_kernel(GemmArgs g, int tiles_m, int tiles_n) {
  gemm_mfma_tile<BM, BN, WGM, WGN, NS, AKS, BKS, BK, CS, KT, SEG, PACK>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.z);
}

// Whether a product of several K segments takes the variant whose cursor looks for a segment's end at every k-tile: where
// padding each segment to whole turns of a ring of ns would run more turns than padding their sum.  (The same turns: the
// cheaper cursor.  No bit depends on it: k-tiles of zeros add nothing.)
// Tiles of which a unit holds one workgroup only: nothing else there hides a k-tile of zeros.  The gradient of the
// attention's input, three segments of the width, us alone with padded segments -> without: 256x128 1024 wide, 8192 rows (54
// k-tiles -> 48) 49.6 -> 47.2, 832 wide (45 -> 39) 40.1 -> 37.0; 128x128 in five stages 1024 wide, 4096 rows (60 -> 50) 33.3
// -> 30.8.  Whole iterations: 832 wide 6154 -> 6124, 704 wide 4861 -> 4835, 1024 wide on 64 units (five stages) 4593 -> 4578.
// The smaller tiles gain alone (64x64, 320 wide, 4096 rows, 24 -> 16: 10.3 -> 8.7) and nothing or less in an iteration,
// where they find the code of one more kernel cold: 320 wide, 4096 rows 1407 / 1407, 318 rows 2042 -> 2068; 128x64, 832
// wide, 2048 rows 2241 -> 2251.
inline bool packs(const GemmArgs& g, int ns, int bk) {
  if (g.K == g.kseg_len) return false;
  const int seg_tiles = (g.kseg_len + bk - 1) / bk, nseg = g.K / g.kseg_len;
  return nseg * ((seg_tiles + ns - 1) / ns) > (nseg * seg_tiles + ns - 1) / ns;
}

template <int BM, int BN, int WGM, int WGN, int NS, bool AKS, bool BKS, int BK, bool PACK, bool CS, bool KT, bool SEG>
static hipError_t launch_kernel(const GemmArgs& g, const GemmLaunch& l) {
  typedef GemmTile<BM, BN, WGM, WGN, NS, AKS, BKS, BK, KT, SEG> CFG;
  if (l.plan) {
    const int seg_tiles = (g.kseg_len + BK - 1) / BK, nseg = g.K / g.kseg_len;
    *l.plan = GemmPlan{BM, BN, BK, PACK ? (nseg * seg_tiles + NS - 1) / NS * NS : nseg * ((seg_tiles + NS - 1) / NS * NS), CFG::NW, NS};
    return hipSuccess;
  }
  auto kern = gemm_mfma_kernel<BM, BN, WGM, WGN, NS, AKS, BKS, BK, CS, KT, SEG, PACK>;
  // once per instantiation, whichever host thread comes first (initialisation of a function-local static is
  // thread-safe)
  static const hipError_t attr_rc = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                        (int)CFG::LDS_BYTES);
  if (attr_rc != hipSuccess) return attr_rc;
  int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
  dim3 grid(tiles_m * tiles_n, 1, g.batch);
  hipLaunchKernelGGL(kern, grid, dim3(CFG::NT), CFG::LDS_BYTES, l.st, g, tiles_m, tiles_n);
  return hipGetLastError();
}

// packed: the same layout's launches with PACK, which are compiled on their own (NULL where these are they)
template <int BM, int BN, int WGM, int WGN, int NS, bool AKS, bool BKS, int BK, bool PACK, bool CS = false, bool KT = false, bool SEG = false>
static hipError_t launch_mfma(const GemmArgs& g, const GemmLaunch& l, LaunchMfma packed) {
  // (the sums of SEG's segments are kept apart: each one starts a turn)
  constexpr bool can_pack = !SEG && !GemmTile<BM, BN, WGM, WGN, NS, AKS, BKS, BK, KT, SEG>::TWO;
  if constexpr (can_pack) {
    if (!PACK && packs(g, NS, BK)) return packed(g, l);
    return launch_kernel<BM, BN, WGM, WGN, NS, AKS, BKS, BK, PACK, CS, KT, SEG>(g, l);
  } else if constexpr (PACK) {
    return hipErrorInvalidValue;   // (no launch asks for it)
  } else {
    return launch_kernel<BM, BN, WGM, WGN, NS, AKS, BKS, BK, PACK, CS, KT, SEG>(g, l);
  }
}

}  // namespace dapple
