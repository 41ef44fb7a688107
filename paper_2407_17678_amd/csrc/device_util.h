// Internal device-side helpers for the gfx950 kernels: MFMA fragment types, the LDS tile that a
// 64-row bf16 chunk is staged in (direct global -> LDS loads, row and transposed fragment reads);
// with the workgroup -> tile mappings (tile_map.h).
//
// Fragment conventions of v_mfma_f32_32x32x16_bf16 (D = A x B + C, 64 lanes, half = lane / 32):
//   A (32 x 16): lane holds row (lane % 32), the 8 k-values of its half.
//   B (16 x 32): lane holds column (lane % 32), the 8 k-values of its half.
//   C/D (32 x 32, 16 floats): lane holds column (lane % 32); register r is row
//        8*(r/4) + 4*half + (r%4).
// The contraction index may be permuted freely as long as A and B agree, which is what lets a
// C-layout tile be fed back as a B operand without moving data between lanes: registers
// 8u..8u+7 of a C tile are, for the lane's half, the rows {16u + 4*half + 0..3,
// 16u + 8 + 4*half + 0..3}; the matching A operand is fetched from LDS in exactly that order
// (see DmaTile::tr_base).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "tile_map.h"

namespace s2 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// v_mfma_f32_16x16x32_bf16 (g = lane / 16):
//   A (16 x 32): lane holds row (lane % 16), the 8 k-values of its g.  B (32 x 16): column (lane % 16), likewise.
//   C/D (16 x 16, 4 floats): lane holds column (lane % 16); register r is row 4 * g + r.
// Two C tiles one below the other (32 rows) are, as a B operand of 32 k-values, four registers each: the lane's k-values are
// rows {4 * g + 0..3, 16 + 4 * g + 0..3}, and ChunkTile::tr_lane fetches the matching A operand in that order.
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// x of this lane combined with x of the lane 32 positions away (the other half of the wavefront).
// v_permlane32_swap exchanges the upper half of one register with the lower half of another: fed
// the same value twice it leaves one register holding the lower half's values in both halves and
// the other the upper half's, so no trip through LDS (and no wait on the LDS counter) is needed.
// Written as inline assembly: with this compiler the builtin's two results come back as one and
// the same register.  The s_nop covers the wait states the instruction needs after a VALU write of
// its operands (the compiler cannot see into the assembly to add them).
__device__ __forceinline__ void swap_halves(float x, float& lo, float& hi) {
  lo = x;
  hi = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
}
__device__ __forceinline__ float max_halves(float x) {
  float a, b;
  swap_halves(x, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float sum_halves(float x) {
  float a, b;
  swap_halves(x, a, b);
  return a + b;
}

// The same with the lane 16 positions away (v_permlane16_swap exchanges the odd rows of 16 lanes of one register with the even
// rows of another), and so over the four lanes that hold one column of a 16x16 tile.
__device__ __forceinline__ void swap_rows(float x, float& even, float& odd) {
  even = x;
  odd = x;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(even), "+v"(odd));
}
__device__ __forceinline__ float max_rows(float x) {
  float a, b;
  swap_rows(x, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float sum_rows(float x) {
  float a, b;
  swap_rows(x, a, b);
  return a + b;
}
__device__ __forceinline__ float sum_groups(float x) { return sum_rows(sum_halves(x)); }

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
// x of a lane of the neighbouring group of M lanes (M = 1, 2, 4, 8), where x is the same in all M lanes of a group: the
// value of lane ^ M, by a lane permutation that an addition takes along instead of a round through the LDS.
template <int M>
__device__ __forceinline__ float of_neighbour(float x) {
  return dpp<M == 1 ? 0xB1 : M == 2 ? 0x4E : M == 4 ? 0x141 : 0x140>(x);  // quad_perm 1032, 2301; half row, row reversed
}

// ---------------------------------------------------------------------------------------------
// DmaTile: a 64-row x D bf16 chunk kept row-major in LDS and filled by direct global -> LDS loads
// (global_load_lds_dwordx4: no staging registers, no LDS store instructions).  Both operand
// forms are read from this one tile: row fragments with 16-byte reads (k = feature) and
// transposed fragments with the LDS transpose read ds_read_b64_tr_b16 (k = token).
//
// Row stride is 76 dwords for D = 128 and 52 dwords for D = 64: measured on gfx950, these are
// strides at which both the 16-byte row reads (32 consecutive rows, the two wavefront halves 16
// bytes apart) and the transpose reads (groups of 16 lanes covering 4 rows x 32 bytes) run at the
// conflict-free rate.  Both tile sizes are whole multiples of the 1024 bytes one wavefront-wide
// direct load fills.
//
// Direct loads write LDS at (wave-uniform base) + 16 * lane, so LDS position decides which global
// address a lane fetches: position p holds row p / stride, 16-byte piece (p % stride) / 16; lanes
// that fall on the pad pieces at the end of a row fetch something harmless (nothing reads the
// padding).
//
// ds_read_b64_tr_b16, within each group of 16 lanes: lane 4e+q supplies the address of 4
// consecutive bf16 (row e of a 4 x 16 block, piece q); lane i receives element i of rows 0..3.
// So a group pointed at tokens t..t+3, features f..f+15 hands lane i the four tokens of feature
// f+i: exactly the k-order of half a C-layout B operand (see the top of this file).
// ---------------------------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));

// Byte address inside LDS of a pointer to __shared__ memory.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// One wavefront-wide direct load: lane i fetches `bytes` (16 or 4) from its own global address
// into LDS at lds_base + bytes * i.  lds_base must be wave-uniform (it goes through M0).
// Written as inline assembly on purpose: the compiler then does not track these loads and so does
// not make unrelated LDS reads wait for a prefetch in flight; the kernels wait for them explicitly
// (wait_all_loads) before the barrier that publishes a stage.  Untracked loads only make the
// compiler's own vmcnt waits more conservative, never less (the counter retires in order).
// The global address is a wave-uniform base (scalar registers) plus a per-lane unsigned 32-bit
// byte offset, so a lane spends one register per load and no 64-bit address arithmetic.
// The s_nop is the wait state a scalar write of M0 needs before an instruction that reads it (the
// compiler would add it for its own code; it does not look inside inline assembly).  M0 is named
// as clobbered so that the compiler does not expect a value of its own to survive there (it warns
// that M0 is a reserved register; the clobber is honoured all the same).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const void* gbase, uint32_t byte_off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(byte_off), "s"(gbase), "s"(lds_base)
               : "memory", "m0");
}
// Two or three loads that share one M0 value.  The instruction's immediate offset is added to the
// global address AND to the LDS address, so loads whose LDS targets differ by less than 4 KiB need only
// one scalar write of M0 (and one wait state) between them; the caller takes the immediate back
// out of the lane's global offset.
template <int I0, int I1>
__device__ __forceinline__ void dma16_group(const void* gbase, uint32_t lds_base, uint32_t o0, uint32_t o1) {
  static_assert(I0 >= 0 && I1 < 4096, "twelve bits");
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %2, %0 offset:%4\n\tglobal_load_lds_dwordx4 %3, %0 offset:%5"
               ::"s"(gbase), "s"(lds_base), "v"(o0), "v"(o1), "n"(I0), "n"(I1)
               : "m0");
}
template <int I0, int I1, int I2>
__device__ __forceinline__ void dma16_group(const void* gbase, uint32_t lds_base, uint32_t o0, uint32_t o1, uint32_t o2) {
  static_assert(I0 >= 0 && I2 < 4096, "twelve bits");
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %0 offset:%5\n\t"
               "global_load_lds_dwordx4 %3, %0 offset:%6\n\tglobal_load_lds_dwordx4 %4, %0 offset:%7"
               ::"s"(gbase), "s"(lds_base), "v"(o0), "v"(o1), "v"(o2), "n"(I0), "n"(I1), "n"(I2)
               : "m0");
}
#pragma clang diagnostic pop

template <int D>
struct DmaTile {
  static constexpr int ROWS = 64;
  static constexpr int kStride = (D == 128) ? 152 : 104;  // elements
  static constexpr int kInstr = (ROWS * kStride * 2 + 1023) / 1024;  // wavefront-wide loads per tile
  static constexpr int kBytes = kInstr * 1024;            // the last load may run past the last row
  static constexpr int kElems = kBytes / 2;

  // lane-dependent part of a transposed fragment's address (elements): features 32*ft + lane%32 of 16 tokens in C-layout k order
  __device__ static __forceinline__ int tr_base(int lane) {
    const int g = lane >> 4, e = (lane & 15) >> 2, q = lane & 3;
    return (4 * (g >> 1) + e) * kStride + 16 * (g & 1) + 4 * q;
  }
};

// ---------------------------------------------------------------------------------------------
// ChunkTile: the tile that goes with the 16x16x32 MFMA.  Its fragments are read as 16 rows x 64 bytes (k = feature) or, by the
// transpose read, 16 rows x 32 bytes, and for these one row stride serves both: 72 dwords (D = 128) or 40 (D = 64), 8 modulo 32.  Measured on
// gfx950, eight wavefronts on a compute unit, cycles an instruction (row reads, transpose reads): 72 dwords 2.0 and 2.5, 76 dwords 4.0 and 3.7, 64
// dwords 16 and 12; the same at 40 and 52.  (The 32x32x16 fragments at DmaTile's 76: 2.0 and 3.7.)
// ---------------------------------------------------------------------------------------------
template <int D>
struct ChunkTile {
  static constexpr int kStride = (D == 128) ? 144 : 80;  // elements
  static constexpr int RB = 2 * kStride;                 // bytes
  static constexpr int kBytes = 64 * RB;                 // a whole number of wavefront-wide loads
  static constexpr int kElems = kBytes / 2;
  // Row fragment: 16-row tile m, features 32 * kk + 8 * g .. + 7 of row lane % 16, at row_lane(lane) + row_off(m, kk)
  __device__ static __forceinline__ uint32_t row_lane(int lane) { return (lane & 15) * RB + 16 * (lane >> 4); }
  static constexpr int row_off(int m, int kk) { return 16 * m * RB + 64 * kk; }
  // Transposed fragment: feature 16 * ft + lane % 16 of the rows {4 * g + 0..3, 16 + 4 * g + 0..3} of 32-row slab u: two transpose
  // reads (see above) at tr_lane(lane) + tr_off(u, ft), the second 16 rows further on
  __device__ static __forceinline__ uint32_t tr_lane(int lane) { return (4 * (lane >> 4) + ((lane & 15) >> 2)) * RB + 8 * (lane & 3); }
  static constexpr int tr_off(int u, int ft) { return 32 * u * RB + 32 * ft; }
};

// ---------------------------------------------------------------------------------------------
// PieceTile: how the four wavefronts of a workgroup fill a 64-row tile by pieces of 16 rows, one
// piece each.  Sixteen padded rows are 4864 bytes (DmaTile, D = 128) or 3328 (64), 4608 or 2560 (ChunkTile), so a piece is
// some whole wavefront-wide loads and one more that ends where the piece ends and fetches the 256 to
// 768 bytes before its remainder a second time (the same bytes to the same place).  The four pieces
// are then back to back - the tile looks exactly as if it had been filled front to back - and where
// each piece comes from is up to the wavefront that fetches it: one scalar row number.  For mask
// blocks of 64 or 128 tokens the pieces are consecutive; for 16- and 32-token blocks a chunk is
// gathered from whatever blocks come next in the tile's list, at no cost per lane.
// ---------------------------------------------------------------------------------------------
template <int D, class TILE = DmaTile<D>>
struct PieceTile {
  static constexpr int kStride = TILE::kStride;         // elements
  static constexpr int kRows = 16;
  static constexpr int kBytes = kRows * kStride * 2;
  static constexpr int kLoads = (kBytes + 1023) / 1024; // 5 / 4 (DmaTile), 5 / 3 (ChunkTile)
  static constexpr int kGroups = kLoads == 3 ? 1 : 2;   // 3 + 2 / 2 + 2 / 3 loads to a write of M0
  static constexpr uint32_t kBias = 4096;
  // where load n starts in the piece: the immediate it is issued with
  __host__ __device__ static constexpr int imm(int n) { return n + 1 < kLoads ? 1024 * n : kBytes - 1024; }
  static_assert(imm(kLoads - 1) < 4096 && kBytes % 16 == 0, "immediates of twelve bits");

  // Byte offset of each of this lane's loads from the piece's first row, plus kBias, minus the
  // immediate (which the instruction adds to the LDS address and to the global one).
  struct Plan {
    uint32_t goff[kLoads];
  };
  __device__ static __forceinline__ Plan plan(int64_t row_stride, int lane) {
    Plan pl;
#pragma unroll
    for (int n = 0; n < kLoads; ++n) {
      const int pos = imm(n) + lane * 16;
      const int row = pos / (kStride * 2);
      int col = (pos - row * kStride * 2) / 16;
      if (col >= D / 8) col -= D / 8;       // row padding: fetches a part of the row again, nothing reads it
      pl.goff[n] = (uint32_t)(row * row_stride * 2) + 16 * col + kBias - imm(n);
    }
    return pl;
  }
  // Group G of the loads of this wavefront's piece into `tile`.  gbase_biased: address of the piece's
  // first row minus kBias bytes.
  template <int G>
  __device__ static __forceinline__ void issue(const Plan& pl, const void* gbase_biased, const uint16_t* tile, int wave) {
    const uint32_t lds = lds_addr(tile) + wave * kBytes;
    if constexpr (kLoads != 4 && G == 0)
      dma16_group<imm(0), imm(1), imm(2)>(gbase_biased, lds, pl.goff[0], pl.goff[1], pl.goff[2]);
    else if constexpr (G == 0)
      dma16_group<imm(0), imm(1)>(gbase_biased, lds, pl.goff[0], pl.goff[1]);
    else
      dma16_group<imm(kLoads - 2), imm(kLoads - 1)>(gbase_biased, lds, pl.goff[kLoads - 2], pl.goff[kLoads - 1]);
  }
  // Limits a plan to pieces of which only the first `rows_valid` (>= 1) rows exist: no lane then reads
  // past the last of them (later rows come out as copies of parts of it; nothing may use them).  A plan
  // limited once can be limited again to fewer rows.
  __device__ static __forceinline__ void limit(Plan& pl, int rows_valid, int64_t row_stride) {
    const uint32_t last = (uint32_t)((rows_valid - 1) * row_stride * 2) + 2 * D - 16 + kBias;
#pragma unroll
    for (int n = 0; n < kLoads; ++n) pl.goff[n] = min(pl.goff[n], last - imm(n));
  }
};

// Everything outstanding (direct loads included) has landed.  This is the builtin, not inline
// assembly, so that the compiler also learns that its own earlier loads (fragments fetched before
// a loop, say) are complete: otherwise it keeps re-waiting for them inside the loop with small
// vmcnt values, and such a wait drains the untracked direct loads that were issued after them.
__device__ __forceinline__ void wait_all_loads() {
  __builtin_amdgcn_s_waitcnt(0);  // vmcnt(0) expcnt(0) lgkmcnt(0)
  asm volatile("" ::: "memory");
}

// At most N of this wavefront's vector-memory operations are still outstanding.  The counter retires in
// issue order, loads and stores alike, so this says that everything issued before the last N has landed
// (direct loads included) without waiting for the last N themselves - stores whose completion nothing
// in the kernel depends on, or loads that are a further step ahead.
template <int N>
__device__ __forceinline__ void wait_loads_but() {
  static_assert(N >= 0 && N < 64, "the counter has six bits");
  // (the caller counts on its last N operations having been issued by now: no store may sink below)
  asm volatile("" ::: "memory");
  // vmcnt in bits 3:0 and 15:14; expcnt (bits 6:4) and lgkmcnt (bits 11:8) at their maxima: no wait
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}

// What this wavefront has asked of the LDS has arrived.
__device__ __forceinline__ void wait_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));  // lgkmcnt(0); vmcnt and expcnt at their maxima: no wait
  asm volatile("" ::: "memory");
}

// Writes 32 rows of results, accumulated as acc[feature tile] with a lane's row in lane % 32, times mul, as
// bf16.  They go out through LDS (`stage`: 32 * (D + 8) elements that are this wavefront's own, so no barrier): a lane
// holds its row's features four at a time, and storing them from there would touch 32 rows per instruction
// with 16 bytes each; read back 16 bytes per lane, row after row, an instruction stores four whole rows.
// GUARD: only the first `rows` rows exist.
template <int D, bool GUARD>
__device__ __forceinline__ void store_rows(const f32x16 (&acc)[D / 32], float mul, uint16_t* stage, uint16_t* base, int64_t row_stride,
                                           int rows, int lane) {
  constexpr int RS = D + 8;  // staging row stride (elements): 8-byte writes of a row group spread over the banks
  static_assert(4 * 32 * RS <= 2 * DmaTile<D>::kElems, "four wavefronts' rows fit two stages");
  const int l32 = lane & 31, half = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[dt][4 * g + e] * mul);
      *reinterpret_cast<bf16x4*>(stage + l32 * RS + 32 * dt + 8 * g + 4 * half) = w;
    }
  constexpr int PPR = D / 8, RPI = 64 / PPR;  // 16-byte pieces per row, rows per instruction
#pragma unroll
  for (int i = 0; i < 32 / RPI; ++i) {
    const int r = RPI * i + lane / PPR, piece = lane % PPR;
    const u32x4 x = *reinterpret_cast<const u32x4*>(stage + r * RS + 8 * piece);
    if (!GUARD || r < rows) *reinterpret_cast<u32x4*>(base + (int64_t)r * row_stride + 8 * piece) = x;
  }
}

// A tile's entry list, held in registers: lane i of the wavefront keeps entry 64*b + i of the
// current batch of 64 entries, and the next batch is fetched one batch ahead, so the main loops
// read their block index with v_readlane instead of waiting on global memory every iteration.
struct EntryList {
  const int32_t* ent;
  int n;         // entries in the list
  int batch;     // which batch of 64 `cur` holds
  int cur, nxt;  // my entry of the current / next batch
  __device__ __forceinline__ void init(const int32_t* list, int count, int lane) {
    ent = list;
    n = count;
    batch = 0;
    cur = lane < n ? ent[lane] : 0;
    nxt = 64 + lane < n ? ent[64 + lane] : 0;
  }
  // entry e (wave-uniform); e never decreases between calls
  __device__ __forceinline__ int get(int e, int lane) {
    if ((e >> 6) != batch) {  // crossed into the next batch
      batch = e >> 6;
      cur = nxt;
      const int i = 64 * (batch + 1) + lane;
      nxt = i < n ? ent[i] : 0;
    }
    return __builtin_amdgcn_readlane(cur, e & 63);
  }
  // entry j of the current or the next batch (64*batch <= j < 64*batch + 128); does not advance
  __device__ __forceinline__ int peek(int j) const {
    return (j >> 6) != batch ? __builtin_amdgcn_readlane(nxt, j & 63) : __builtin_amdgcn_readlane(cur, j & 63);
  }
  // the same without a branch, and 0 past the list's end
  __device__ __forceinline__ int at(int j) const {
    const int a = __builtin_amdgcn_readlane(cur, j & 63), b = __builtin_amdgcn_readlane(nxt, j & 63);
    return (j >> 6) == batch ? a : b;
  }
};

}  // namespace s2
