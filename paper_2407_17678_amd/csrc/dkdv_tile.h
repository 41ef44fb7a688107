// One workgroup's share of the dK/dV launch: a tile of 128 keys (or a part of one), column-stationary - of the launch in bwd_kernel.hip, or
// of that in bwd_merged_kernel.hip, which holds dQ tiles too.
//
// The dK/dV loop is written out fragment by fragment, one slot and two MFMAs each (see sched_util.h): for 32 query rows S, dP, dV and dK one
// after the other, the exponentials under dP, dS = P * dP under dV, each LDS fragment requested three slots ahead of its use through a ring
// that goes on from one half step to the next, across the barrier too: it lies before the last three slots of a step.  Left to the compiler
// every MFMA waited for the read issued right before it, since at 192 registers of accumulators and K / V fragments it keeps no second
// fragment.  Room for the ring comes from what no longer has registers: the row statistics are read straight into the accumulators (S begins at
// -lse / scale, dP at -delta), the lane offsets of the direct loads lie in LDS, and what derives from the lane number is
// formed where it is used.  dK/dV launch, before, with the slots, and with the ring going across the barrier: 1 x 32 heads x 32768 x 128
// 1.980, 1.872, 1.820 ms (2.262, 2.195, 2.157 where it keeps dS), 4 x 32 x 8192 x 64 0.639, 0.625, 0.603 ms.
//
// What bounds it then is power: the chip's clock falls from 2.4 GHz to about 1.6 under it (GRBM_GUI_ACTIVE).  A loop of nothing but
// 32x32x16 MFMAs on random operands sustains 1.75 PFLOP/s at 1.76 GHz, one of 16x16x32 MFMAs 2.06 at 2.07, and with one 16-byte LDS read to 32
// cycles of either 1.59 and 1.81: hence the smaller shape, whose fragments of 16 rows also leave the LDS fewer bank conflicts (ChunkTile).
// Same launches, 32x32x16 and 16x16x32: 1.820 and 1.740 ms (2.157 and 2.070 keeping dS), 4 x 32 x 8192 x 64 603 and 511 us, 3 x 20 x 8192 x
// 64 with 32-token blocks 171 and 152.
#pragma once
#include <hip/hip_runtime.h>

#include "config.h"
#include "device_util.h"
#include "kernels.h"
#include "sched_util.h"

namespace s2 {

// To and from memory that other workgroups, on any XCD, write and read in the same launch: the sc1 bit is
// agent scope, past the caches that the XCDs do not share (what a relaxed atomic of that scope compiles
// to, sixteen bytes at a time).  Base in scalar registers, a lane offset in bytes, an immediate.
template <int OFF>
__device__ __forceinline__ void store_agent(void* base, uint32_t lane_off, f32x4 x) {
  // (the no-op is the wait state a wide store needs before its data registers are written again)
  asm volatile("global_store_dwordx4 %0, %1, %2 offset:%3 sc1\n\ts_nop 0" ::"v"(lane_off), "v"(x), "s"(base), "n"(OFF) : "memory");
}
// sixteen kilobyte-wide loads in flight together, and the wait for them
__device__ __forceinline__ void load_agent16(const void* base, uint32_t lane_off, f32x4 (&x)[16]) {
  const char* b0 = static_cast<const char*>(base);
  asm volatile("global_load_dwordx4 %0, %16, %17 sc1\n\tglobal_load_dwordx4 %1, %16, %17 offset:1024 sc1\n\t"
               "global_load_dwordx4 %2, %16, %17 offset:2048 sc1\n\tglobal_load_dwordx4 %3, %16, %17 offset:3072 sc1\n\t"
               "global_load_dwordx4 %4, %16, %18 sc1\n\tglobal_load_dwordx4 %5, %16, %18 offset:1024 sc1\n\t"
               "global_load_dwordx4 %6, %16, %18 offset:2048 sc1\n\tglobal_load_dwordx4 %7, %16, %18 offset:3072 sc1\n\t"
               "global_load_dwordx4 %8, %16, %19 sc1\n\tglobal_load_dwordx4 %9, %16, %19 offset:1024 sc1\n\t"
               "global_load_dwordx4 %10, %16, %19 offset:2048 sc1\n\tglobal_load_dwordx4 %11, %16, %19 offset:3072 sc1\n\t"
               "global_load_dwordx4 %12, %16, %20 sc1\n\tglobal_load_dwordx4 %13, %16, %20 offset:1024 sc1\n\t"
               "global_load_dwordx4 %14, %16, %20 offset:2048 sc1\n\tglobal_load_dwordx4 %15, %16, %20 offset:3072 sc1\n\t"
               "s_waitcnt vmcnt(0)"
               : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7]),
                 "=&v"(x[8]), "=&v"(x[9]), "=&v"(x[10]), "=&v"(x[11]), "=&v"(x[12]), "=&v"(x[13]), "=&v"(x[14]), "=&v"(x[15])
               : "v"(lane_off), "s"(b0), "s"(b0 + 4096), "s"(b0 + 8192), "s"(b0 + 12288)
               : "memory");
}

// x stays where AT >= lim (keep_from) or AT < lim (keep_below), else it becomes `gone`.  Written out so that it costs no register but
// its operands: left to itself the compiler keeps the compares of a whole tile at hand, and `gone` over the whole kernel.
// (The no-op is the wait between a vector write of vcc and its use as a select.)
template <int AT>
__device__ __forceinline__ float keep_from(float x, int lim, float gone) {
  asm volatile("v_cmp_ge_i32 vcc, %2, %1\n\ts_nop 1\n\tv_cndmask_b32 %0, %3, %0, vcc" : "+v"(x) : "v"(lim), "n"(AT), "v"(gone) : "vcc");
  return x;
}
template <int AT>
__device__ __forceinline__ float keep_below(float x, int lim, float gone) {
  asm volatile("v_cmp_lt_i32 vcc, %2, %1\n\ts_nop 1\n\tv_cndmask_b32 %0, %3, %0, vcc" : "+v"(x) : "v"(lim), "n"(AT), "v"(gone) : "vcc");
  return x;
}
template <uint32_t BITS>
__device__ __forceinline__ float constant_now() {
  float x;
  asm volatile("v_mov_b32 %0, %1" : "=v"(x) : "n"((int)BITS));
  return x;
}
constexpr uint32_t kNegInfBits = 0xFF800000u;

template <int D>
struct DkvSmem {
  uint16_t q[2][ChunkTile<D>::kElems];
  uint16_t g[2][ChunkTile<D>::kElems];
  struct RowStats {
    float neg_delta[64];
    float neg_lse[64];
  } rs[2];                 // one 512-byte direct load fills both arrays of a stage
  uint32_t goff[PieceTile<D, ChunkTile<D>>::kLoads][64];  // the lane offsets of the direct loads
};

// FINE: mask blocks of 16 or 32 tokens (0: larger ones).  A step's 64 query rows are four pieces of 16
// gathered from the next blocks of the tile's list (entries of single blocks, one bit per mask column of
// the tile), and the tile's 4 or 8 columns are any that are attended by nearly the same rows, so a
// wavefront's 32 keys are one or two columns and what a lane drops of a piece depends on its column.
// (Steps of 32 rows over tiles of adjacent columns, as before, had one stripe column keep three idle ones
// company.)  A 32-row half that none of them attends is left out.  With blocks of 16 a half is two blocks
// and a wavefront two columns: a row that is not a number reaches dK and dV of both columns if either of the
// half's blocks attends either (keeping it from them, by zeros for dS and the other block's rows, was built and
// cost 10 to 18 %: spilled registers at head_dim 128, the selects at 64).
//
// VARLEN: a packed batch of sequences of different lengths.  A key tile's members are columns of
// the whole layout, so the workgroup first drops out if none of them exists in its sequence, skips
// the list entries (query blocks, last first) that lie after the sequence's end, clamps the loads
// of the ragged last chunk and zeroes P and dS for the query rows of it that do not exist.
// STORE: dS, rounded to bf16 as the dK contraction takes it, is also left in the workspace for the dQ
// launch (launch_dq_gemm), 4 KiB per wavefront and step: [32-query half][key][g = lane / 16][8 queries as the lane
// holds them: 4 * g + 0..3, then 16 + 4 * g + 0..3], i.e. each B operand (16 keys) as it is, 1 KiB per store instruction.
template <int D, bool DENSE, int FINE, bool VARLEN = false, bool STORE = false>
__device__ __forceinline__ void dkdv_tile(const AttnParams& p, int wg, unsigned char* smem_raw) {
  typedef ChunkTile<D> Tile;
  typedef PieceTile<D, Tile> Piece;
  constexpr int CH = 64;
  constexpr int KS = D / 32;                                  // 32-feature steps of the S and dP contractions
  constexpr int FT = D / 16;                                  // 16-feature tiles of dK and dV
  constexpr int KK = D / 16;                                  // fragments of each contraction, two MFMAs each
  static_assert(2 * KS == KK && FT == KK, "two 16-row tiles by KS steps; one 32-row slab by FT tiles");
  constexpr int RB = Tile::RB;                                // bytes per tile row
  constexpr int G_OFF = 2 * Tile::kBytes;                     // dO stages lie after the Q stages
  constexpr int kLead = VARLEN ? 2 : 3, kRing = 4;            // (packed batches have no room for three; the same time)
  static_assert((4 * KK) % kRing == 0, "the ring goes on from half to half");
  constexpr int kTr = 2 * KK - kLead;                         // the slot that requests the first transposed fragment
  static_assert(!(DENSE && (FINE || VARLEN)) && !(STORE && (DENSE || FINE || VARLEN)), "forms that exist");
  static_assert(FINE == 0 || FINE == 16 || FINE == 32, "blocks that are gathered");
  constexpr int PPE = FINE == 32 ? 2 : 1, EPC = 4 / PPE;  // FINE: 16-row pieces of a list entry, entries of a step
  DkvSmem<D>& sm = *reinterpret_cast<DkvSmem<D>*>(smem_raw);

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int T = p.kv_tiles.tiles_per_head;
  constexpr bool kSplits = !DENSE && !VARLEN;
  int bh, rank;
  if (!map_workgroup_interleaved(p.key_map, wg, bh, rank)) return;
  const int b = bh / p.by_heads, h = bh - b * p.heads;
  // which part of which tile, in descending length: the parts of the tiles that are cut, then the others
  int part = 0, parts = 1, nth = rank;
  if (kSplits) {
    if (rank < p.split_items) {
      const int code = load_const<int32_t>(p.split_codes + rank);
      nth = code & 0xFFFF;
      part = (code >> 16) & 0xFF;
      parts = code >> 24;
    } else {
      nth = rank - p.split_items + p.split_long;
    }
  }
  const int32_t* const rec = DENSE ? nullptr : p.kv_tiles.col_rec(h, nth);  // (dense: first key tiles are longest)
  const int S = DENSE ? CH : FINE ? FINE : p.block_size;
  const int cpb_sh = S == 128 ? 1 : 0, cpb_m = (1 << cpb_sh) - 1, s_sh = 6 + cpb_sh;  // chunks per list entry; S of one as a shift
  int row_base = 0, N = p.seqlen;
  if (VARLEN) {
    const int lo = load_const<int32_t>(p.cu_seqlens + b), hi = load_const<int32_t>(p.cu_seqlens + b + 1);
    row_base = min(max(lo, 0), p.seqlen);  // whatever the array holds, stay inside the tensors
    N = min(min(max(hi - lo, 0), p.q_rows), p.seqlen - row_base);
  }

  // My 32 keys: kvw0 .. kvw0 + 31, or (blocks of 16) keys 0..15 from kvw0 and 16..31 from kvw1.  A group of keys
  // that does not exist (the layout's last tile, a packed sequence's end) starts at kNoKey.
  constexpr int kNoKey = 1 << 29;
  int kvw0, kvw1, my_member = 0;
  bool wave_active;
  if (DENSE) {
    kvw0 = rank * kBwdBN + wave * 32;
    kvw1 = kvw0 + 16;
    wave_active = kvw0 < N;
  } else {
    const int32_t* mem = rec + 4;
    if (VARLEN) {  // the whole workgroup leaves together when none of its columns is in the sequence
      bool any = false;
      for (int m = 0; m < p.kv_tiles.group; ++m) {
        const int blk = load_const<int32_t>(mem + m);
        any = any || (blk >= 0 && blk * S < N);
      }
      if (!any) return;
    }
    const int sh = FINE == 16 ? 4 : FINE == 32 ? 5 : s_sh;
    my_member = (wave * 32) >> sh;
    const int blk0 = load_const<int32_t>(mem + my_member), blk1 = load_const<int32_t>(mem + ((wave * 32 + 16) >> sh));
    kvw0 = blk0 < 0 ? kNoKey : blk0 * S + ((wave * 32) & (S - 1));
    kvw1 = blk1 < 0 ? kNoKey : blk1 * S + ((wave * 32 + 16) & (S - 1));
    wave_active = FINE == 16 ? min(kvw0, kvw1) < N : kvw0 < N;
  }
  // key of row r (0..31) of mine
  auto key_of = [&](int r) S2_INLINE { return FINE == 16 ? (r < 16 ? kvw0 + r : kvw1 + r - 16) : kvw0 + r; };

  const int64_t q_off = (VARLEN ? row_base * p.q_st : b * p.q_sb) + h * p.q_sh;
  const int64_t kv_off = (VARLEN ? row_base * p.kv_st : b * p.kv_sb) + h * p.kv_sh;
  // minus the bias the grouped direct loads put into their lane offsets
  const char* qb = reinterpret_cast<const char*>(p.q + q_off) - Piece::kBias;
  const char* gb = reinterpret_cast<const char*>(p.d_o + q_off) - Piece::kBias;
  const uint32_t row_bytes = (uint32_t)(2 * p.q_st);  // (api.hip: at most 2^25)
  // packed batch: the row statistics are [heads, rows of the tensors]
  const int64_t stats_off = VARLEN ? (int64_t)h * p.seqlen + row_base : ((int64_t)b * p.heads + h) * N;
  const float* lse_b = p.neg_lse + stats_off;
  const float* delta_b = p.neg_delta + stats_off;

  int ent_lo = 0, n_ent;
  if (DENSE) {
    n_ent = (N - rank * kBwdBN) / kChunk;  // query chunks at or after the tile's first key
  } else {
    ent_lo = load_const<int32_t>(rec + 1);
    n_ent = load_const<int32_t>(rec + 2);
  }
  if (kSplits && parts > 1) {  // my part: so many entries, or (FINE) so many full steps of entries
    const int units = FINE ? (n_ent + EPC - 1) / EPC : n_ent;
    const int u0 = units * part / parts, u1 = units * (part + 1) / parts;
    const int e0 = FINE ? EPC * u0 : u0;
    n_ent = (FINE ? min(EPC * u1, n_ent) : u1) - e0;
    ent_lo += e0;
  }
  // steps: chunks of an entry, or (FINE) as many as the entries' pieces fill
  const int total = FINE ? (n_ent + EPC - 1) / EPC : n_ent << cpb_sh;
  // where this wavefront's dS of step 0 goes: unit 2 * (global step) + wave / 2, its keys' half of it
  uint16_t* ds_wave = nullptr;
  if (STORE)
    ds_wave = p.ds_store + ((int64_t)b * p.ds_units + (((int64_t)ent_lo << cpb_sh) * 2 + (wave >> 1))) * 4096 + (wave & 1) * 2048;
  EntryList list;
  if (!DENSE) list.init(p.kv_tiles.ent + ent_lo, n_ent, lane);
  // K and V fragments (B operands) [32-feature step][16-key tile], lane % 16 = key of the tile; requested while the list is on its way
  bf16x8 kf[KS][2], vf[KS][2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    // (a lane whose key does not exist reads an existing one: every pair of it is masked and nothing is stored)
    const int64_t row = kv_off + (int64_t)min(key_of(16 * nt + (lane & 15)), N - 1) * p.kv_st + 8 * (lane >> 4);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      kf[kk][nt] = *reinterpret_cast<const bf16x8*>(p.k + row + 32 * kk);
      vf[kk][nt] = *reinterpret_cast<const bf16x8*>(p.v + row + 32 * kk);
    }
  }
  // FINE: the entries of step j, in lanes EPC * j % 64 and on (0 after the end of the list: attends nobody)
  auto entries_at = [&](int j) S2_INLINE { return ((EPC * j) >> 6) != list.batch ? list.nxt : list.cur; };
  auto entry = [&](int src, int i) S2_INLINE { return (uint32_t)__builtin_amdgcn_readlane(src, i & 63); };
  // not FINE: first row of step j, and whether my mask column is kept there
  auto chunk_at = [&](int j, int& q0, bool& keep) S2_INLINE {
    if (DENSE) {
      q0 = N - CH - j * CH;  // from the last query chunk down, like the sparse lists
      keep = true;
    } else {
      const uint32_t e = (uint32_t)list.at(j >> cpb_sh);
      q0 = (int)(e >> 16 << s_sh) + ((cpb_m - (j & cpb_m)) << 6);
      keep = (e >> my_member) & 1;
    }
  };

  // FINE: the largest entry whose query block begins before my sequence's end
  const uint32_t last_ent = FINE && VARLEN ? ((uint32_t)((N + FINE - 1) / max(FINE, 1) - 1) << 16) | 0xFFFFu : 0;
  const typename Piece::Plan plan = Piece::plan(p.q_st, lane);
  const uint32_t stats_gap = (uint32_t)((const char*)lse_b - (const char*)delta_b);
  // `ln` is the lane number.  The loop passes a copy the optimiser cannot see through, so that
  // what is derived from it is recomputed each step (a few integer operations) rather than kept in
  // registers across the loop: this kernel has no registers to spare, and a spilled constant costs
  // a wait for all outstanding loads when it is fetched back.
  const int wave_of = wave;
  auto issue_chunk = [&](const typename Piece::Plan& plan, int j, int buf, int ln) S2_INLINE {
    int q0 = 0, src = 0, row;
    const int wave = __builtin_amdgcn_readfirstlane(wave_of);  // (into a scalar register again: the compiler may hold it in a vector one)
    if constexpr (FINE) {
      src = entries_at(j);
      row = (int)(entry(src, EPC * j + wave / PPE) >> 16) * FINE + 16 * (wave % PPE);
    } else {
      bool keep;
      chunk_at(j, q0, keep);
      row = q0 + 16 * wave;
    }
    // Ragged end of a packed sequence: rows past it fetch parts of its last row instead (a list need
    // not be in descending order, so a piece that lies wholly after the end can turn up anywhere in
    // it: nothing uses it).
    typename Piece::Plan pl = plan;
    if (VARLEN && row + 16 > N) {
      row = min(row, N - 1);
      Piece::limit(pl, N - row, p.q_st);
    }
    const uint64_t at = (uint64_t)(uint32_t)row * row_bytes;
    const char *qg = qb + at, *gg = gb + at;
    static_for<Piece::kGroups>([&](auto gc) S2_INLINE { Piece::template issue<decltype(gc)::value>(pl, qg, sm.q[buf], wave); });
    static_for<Piece::kGroups>([&](auto gc) S2_INLINE { Piece::template issue<decltype(gc)::value>(pl, gg, sm.g[buf], wave); });
    // 64 floats of each array: lanes 0..15 fetch delta, lanes 16..31 lse, 16 bytes each, in one direct load.
    // (Where a packed sequence ends inside a piece the rest of it comes from the slack of the workspace
    // or from the next rows: nothing uses it.)
    if (wave == 3) {
      uint32_t off;
      if constexpr (FINE) {
        const int pc = (ln >> 2) & 3;
        int r[4];  // first row of each piece
#pragma unroll
        for (int n = 0; n < 4; ++n) r[n] = (int)(entry(src, EPC * j + n / PPE) >> 16) * FINE + 16 * (n % PPE);
        int pr = pc == 0 ? r[0] : pc == 1 ? r[1] : pc == 2 ? r[2] : r[3];
        if (VARLEN) pr = min(pr, N - 1);
        off = 4 * pr + 16 * (ln & 3) + ((ln & 16) ? stats_gap : 0u);
      } else {
        off = 16 * (ln & 15) + ((ln & 16) ? stats_gap : 0u) + 4 * (VARLEN && q0 >= N ? 0 : q0);
      }
      if (ln < 32) dma16(delta_b, off, lds_addr(&sm.rs[buf]));
    }
  };
  // first step: a packed sequence skips the leading entries, query blocks that lie after its end (most
  // lists start at the layout's last row; such blocks further on are walked without being used)
  int it0 = 0;
  if (VARLEN) {
    int e = 0;
    for (; e < n_ent; e += 64) {
      (void)list.get(e, lane);
      const uint64_t in = __ballot(e + lane < n_ent && (int)((uint32_t)list.cur >> 16) * S < N);
      if (in) {
        e += __builtin_ctzll(in);
        break;
      }
    }
    e = min(e, n_ent - 1);  // (a key of the sequence is attended by its own block at least)
    (void)list.get(e, lane);
    it0 = FINE ? e / EPC : e << cpb_sh;
  }
  if (!kSplits || total > 0) issue_chunk(plan, it0, it0 & 1, lane);  // (where a head's tile is short for its rank a part may be empty)

  // dK and dV, transposed [16-feature tile][16-key tile]: lane % 16 = key, register r = feature 4 * (lane / 16) + r
  f32x4 acc_dk[FT][2], acc_dv[FT][2];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) acc_dk[ft][nt] = acc_dv[ft][nt] = f32x4{};
  const float c = p.p_scale_log2e;
  if (wave == 0) {
#pragma unroll
    for (int n = 0; n < Piece::kLoads; ++n) sm.goff[n][lane] = plan.goff[n];
  }

  // The walk is one sequence of half steps of 32 query rows: half qt (up to qt1 - 1) of step it, whose first row is q0 (not FINE) or
  // whose entries are in ents.
  uint32_t ents[EPC] = {};
  int it = __builtin_amdgcn_readfirstlane(it0) - 1, qt = 0, qt1 = 0, q0 = 0, stores = 0;  // stores: dS stores since the last direct loads
  bool refill = false;  // the chunk of the step after this one has yet to be requested, into the other stage
  auto request_next = [&]() S2_INLINE {
    refill = false;
    stores = 0;
    if (it + 1 >= total) return;
    const int ln = lane_now();
    typename Piece::Plan pl;
#pragma unroll
    for (int n = 0; n < Piece::kLoads; ++n) pl.goff[n] = sm.goff[n][ln];
    issue_chunk(pl, it + 1, (it + 1) & 1, ln);
  };
  // opens step it: finds the halves that hold something for my keys
  auto open_step = [&]() S2_INLINE {
    // keeps the entry window moving (entries of this step on)
    if (!DENSE) (void)list.get(FINE ? EPC * it : it >> cpb_sh, lane_now());
    refill = true;
    int lo = 0, hi = 0;
    if constexpr (FINE) {
      // which pieces of the step attend keys of mine, from every lane's entry at once
      const int src = entries_at(it);
#pragma unroll
      for (int i = 0; i < EPC; ++i) ents[i] = entry(src, EPC * it + i);
      uint64_t any = __ballot(FINE == 32 ? ((src >> wave) & 1) != 0 : ((src >> (2 * wave)) & 3) != 0);
      if (VARLEN) any &= __ballot((uint32_t)src <= last_ent);
      const uint32_t on4 = (uint32_t)(any >> ((EPC * it) & 63));
      lo = (on4 & (FINE == 32 ? 1 : 3)) ? 0 : 1;
      hi = !wave_active ? 0 : (on4 & (FINE == 32 ? 2 : 12)) ? 2 : 1;
    } else {
      bool keep;
      chunk_at(it, q0, keep);
      lo = q0 + 31 < kvw0 ? 1 : 0;  // (every query of the half lies before my keys)
      hi = !wave_active || !keep || q0 + CH - 1 < kvw0 ? 0 : 2;
      if (VARLEN) hi = q0 >= N ? 0 : q0 + 32 >= N ? min(hi, 1) : hi;  // ... or after the end of my sequence
    }
    qt = __builtin_amdgcn_readfirstlane(lo);
    qt1 = __builtin_amdgcn_readfirstlane(hi);
  };
  // Goes on to the next half (false: there is none), through the barrier where that is in another step: by then the next chunk has
  // landed and every wavefront has read what it needs of this one.  Exactly one barrier a step, whatever I have to do in it.
  auto next_half = [&]() S2_INLINE {
    if (++qt < qt1) return true;
    do {
      // (this step's dS stores, issued after its loads, may stay in flight)
      if (STORE && stores == 4)
        wait_loads_but<4>();
      else if (STORE && stores == 2)
        wait_loads_but<2>();
      else
        wait_loads_but<0>();
      wait_lds();
      __syncthreads();
      it = __builtin_amdgcn_readfirstlane(it + 1);
      if (it >= total) return false;
      open_step();
      if (qt >= qt1) request_next();
    } while (qt >= qt1);
    return true;
  };
  wait_all_loads();
  bool more = next_half();  // (after the last half the loop still requests fragments, from inside the stages, that nothing uses)
  if (more) {
    uint32_t row_a, tr_a, st_a;
    // where the lane finds its rows of the half's tiles and statistics
    auto aim_rows = [&]() S2_INLINE {
      const int ln = lane_now(), buf = it & 1;
      row_a = lds_addr(sm.q[0]) + buf * (uint32_t)Tile::kBytes + qt * 32 * RB + Tile::row_lane(ln);
      st_a = lds_addr(&sm.rs[0]) + buf * (uint32_t)sizeof(sm.rs[0]) + 128 * qt + 16 * (ln >> 4);
      asm volatile("" : "+v"(row_a), "+v"(st_a));
    };
    auto aim_tr = [&]() S2_INLINE {
      tr_a = lds_addr(sm.q[0]) + (it & 1) * (uint32_t)Tile::kBytes + qt * 32 * RB + Tile::tr_lane(lane_now());
      asm volatile("" : "+v"(tr_a));
    };
    bf16x8 fr[kRing];
    // [16-row tile m][16-key tile nt]: lane % 16 = key, register r = row 4 * (lane / 16) + r
    f32x4 s[2][2], dp[2][2];    // S, then P in place; dP, then dS in place
    f32x4 st_s[2], st_d[2];     // what S and dP begin with: the statistics of the lane's rows
    // fragment f of a half, in the order the MFMAs use them; those after the last are the first of the next half
    auto frag_load = [&](auto fc) S2_INLINE {
      constexpr int f = decltype(fc)::value;
      u32x4 x;
      if constexpr (f < KK)
        x = lds_read16(row_a, Tile::row_off(f & 1, f >> 1));
      else if constexpr (f < 2 * KK)
        x = lds_read16(row_a, G_OFF + Tile::row_off((f - KK) & 1, (f - KK) >> 1));
      else if constexpr (f < 3 * KK)
        x = lds_read_tr(tr_a, G_OFF + Tile::tr_off(0, f - 2 * KK), 2 * RB);
      else if constexpr (f < 4 * KK)
        x = lds_read_tr(tr_a, Tile::tr_off(0, f - 3 * KK), 2 * RB);
      else
        x = lds_read16(row_a, Tile::row_off((f - 4 * KK) & 1, (f - 4 * KK) >> 1));
      fr[f % kRing] = __builtin_bit_cast(bf16x8, x);
    };
    auto stats_load = [&](int m) S2_INLINE {
      st_s[m] = lds_read_f32x4(st_a, 256 + 64 * m);
      st_d[m] = lds_read_f32x4(st_a, 64 * m);
    };
    aim_rows();
    stats_load(0);
    stats_load(1);
    static_for<kLead>([&](auto fc) S2_INLINE { frag_load(fc); });
    request_next();
    do {
      // row of tile m's first row, and (FINE) the list entry it comes from
      int row[2] = {q0 + 32 * qt, q0 + 32 * qt + 16};
      uint32_t ent[2] = {~0u, ~0u};
      if constexpr (FINE) {
        ent[0] = qt ? ents[EPC / 2] : ents[0];
        ent[1] = FINE == 32 ? ent[0] : qt ? ents[EPC - 1] : ents[1];
        row[0] = (int)(ent[0] >> 16) * FINE;
        row[1] = FINE == 32 ? row[0] + 16 : (int)(ent[1] >> 16) * FINE;
      }
      // some pair of the half is dropped: its query lies before its key or (blocks of 16) my column does not keep the piece
      bool masked = min(row[0], row[1]) < (FINE == 16 ? max(kvw0, kvw1) + 15 : kvw0 + 31);
      if (FINE == 16) masked = masked || (((ent[0] & ent[1]) >> (2 * wave)) & 3) != 3;
      const bool ragged = VARLEN && max(row[0], row[1]) + 16 > N;
      u32x4 pb[2], dsb[2];  // P and dS as B operands [16-key tile]
      // element x (0..15) of s or dp, in the order of the B operands: tile [(x >> 2) & 1][x >> 3], register x & 3
      auto elem = [](f32x4 (&a)[2][2], int x) S2_INLINE -> float { return a[(x >> 2) & 1][x >> 3][x & 3]; };
      auto pack_operand = [&](f32x4 (&a)[2][2], int nt) S2_INLINE {
        return u32x4{pack2(elem(a, 8 * nt), elem(a, 8 * nt + 1)), pack2(elem(a, 8 * nt + 2), elem(a, 8 * nt + 3)),
                     pack2(elem(a, 8 * nt + 4), elem(a, 8 * nt + 5)), pack2(elem(a, 8 * nt + 6), elem(a, 8 * nt + 7))};
      };
      // VARLEN: `gone` where a row lies past the sequence's end
      auto drop_past_end = [&](auto gone, f32x4 (&a)[2][2]) S2_INLINE {
        const float drop = constant_now<decltype(gone)::value>();
        const int g4 = 4 * (lane_now() >> 4);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int left = N - row[m] - g4;
          S2_FENCE();
#pragma unroll
          for (int nt = 0; nt < 2; ++nt)
            static_for<4>([&](auto rc) S2_INLINE { a[m][nt][decltype(rc)::value] = keep_below<decltype(rc)::value>(a[m][nt][decltype(rc)::value], left, drop); });
        }
      };
      S2_FENCE();
      static_for<4 * KK>([&](auto nc) S2_INLINE {
        constexpr int n = decltype(nc)::value;
        if constexpr (n == kTr) aim_tr();
        // every fragment of this half is requested: on to the next one
        if constexpr (n + kLead == 4 * KK) {
          more = next_half();
          aim_rows();
        }
        frag_load(std::integral_constant<int, n + kLead>{});
        if constexpr (n == 4 * KK - 1) {
          if (refill) request_next();  // (after the first fragments of the step, which its MFMAs wait for)
        }
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          if constexpr (n < KK) {
            constexpr int m = n & 1, kk = n >> 1;
            s[m][nt] = mfma16(fr[n % kRing], kf[kk][nt], kk == 0 ? st_s[m] : s[m][nt]);
          } else if constexpr (n < 2 * KK) {
            constexpr int m = n & 1, kk = (n - KK) >> 1;
            dp[m][nt] = mfma16(fr[n % kRing], vf[kk][nt], kk == 0 ? st_d[m] : dp[m][nt]);
          } else if constexpr (n < 3 * KK) {
            acc_dv[n - 2 * KK][nt] = mfma16(fr[n % kRing], __builtin_bit_cast(bf16x8, pb[nt]), acc_dv[n - 2 * KK][nt]);
          } else {
            acc_dk[n - 3 * KK][nt] = mfma16(fr[n % kRing], __builtin_bit_cast(bf16x8, dsb[nt]), acc_dk[n - 3 * KK][nt]);
          }
        }
        constexpr int M0 = KK + 1, D0 = 2 * KK + 1;
        if constexpr (n == M0) {
          if (masked) {
            const int ln = lane_now(), l16 = ln & 15, g4 = 4 * (ln >> 4);
            const float drop = constant_now<kNegInfBits>();
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
              for (int nt = 0; nt < 2; ++nt) {
                const int key0 = FINE == 16 && nt ? kvw1 : kvw0 + 16 * nt;
                if (FINE == 16 && !((ent[m] >> (2 * wave + nt)) & 1)) {  // the tile is a block my column does not keep
                  s[m][nt] = f32x4{drop, drop, drop, drop};
                } else if (FINE != 16 || row[m] < key0 + 15) {
                  const int lim = key0 + l16 - row[m] - g4;
                  S2_FENCE();
                  static_for<4>([&](auto rc) S2_INLINE { s[m][nt][decltype(rc)::value] = keep_from<decltype(rc)::value>(s[m][nt][decltype(rc)::value], lim, drop); });
                }
              }
          }
          if (ragged) drop_past_end(std::integral_constant<uint32_t, kNegInfBits>{}, s);
        }
        // P: scaled in slots M0 .., the exponential a slot behind, all of it before dV begins
        constexpr int NP = KK - 2;
        auto upto = [](int i) { return i < 0 ? 0 : i >= NP ? 16 : (16 * i + NP - 1) / NP; };
        if constexpr (n >= M0 && n < M0 + NP) {
#pragma unroll
          for (int x = upto(n - M0); x < upto(n - M0 + 1); ++x) s[(x >> 2) & 1][x >> 3][x & 3] *= c;
        }
        if constexpr (n > M0 && n <= M0 + NP) {
#pragma unroll
          for (int x = upto(n - M0 - 1); x < upto(n - M0); ++x) s[(x >> 2) & 1][x >> 3][x & 3] = fast_exp2(s[(x >> 2) & 1][x >> 3][x & 3]);
        }
        static_assert(M0 + NP == 2 * KK - 1, "P is complete in the slot before dV begins");
        if constexpr (n == 2 * KK - 1) {
          pb[0] = pack_operand(s, 0);
          pb[1] = pack_operand(s, 1);
        }
        // dS under dV
        constexpr int ND = KK - 1;
        auto dupto = [](int i) { return i >= ND ? 16 : (16 * i + ND - 1) / ND; };
        if constexpr (n >= D0 && n < D0 + ND) {
#pragma unroll
          for (int x = dupto(n - D0); x < dupto(n - D0 + 1); ++x) dp[(x >> 2) & 1][x >> 3][x & 3] *= s[(x >> 2) & 1][x >> 3][x & 3];
          asm volatile("" : "+v"(dp[0][0]), "+v"(dp[0][1]), "+v"(dp[1][0]), "+v"(dp[1][1]));
        }
        if constexpr (n == 3 * KK - 1) {
          if (ragged) drop_past_end(std::integral_constant<uint32_t, 0>{}, dp);  // (their statistics are not their own)
          dsb[0] = pack_operand(dp, 0);
          dsb[1] = pack_operand(dp, 1);
          if constexpr (STORE) {
            const uint32_t off = 64u * (lane_now() & 15) + 16u * (lane_now() >> 4);
            unsigned char* const unit = reinterpret_cast<unsigned char*>(ds_wave + (int64_t)it * 8192 + 1024 * qt);
            // non-temporal: written once here and read by a later launch, it should not push the Q / dO
            // blocks this kernel re-reads out of L2
            __builtin_nontemporal_store(dsb[0], reinterpret_cast<u32x4*>(unit + off));
            __builtin_nontemporal_store(dsb[1], reinterpret_cast<u32x4*>(unit + 1024 + off));
            stores += 2;
          }
        }
        // the next half's statistics, where its contractions begin
        if constexpr (n == 4 * KK - kLead) stats_load(0);
        if constexpr (n == 4 * KK - kLead + 1) stats_load(1);
        S2_FENCE();
      });
    } while (more);
  }

  if (kSplits && parts > 1) {
    // This is a part of a tile: leave my sums in memory, and if the other parts have done so already add
    // all of them up, in the order of the parts, and go on with the result.
    constexpr int kTiles = FT;                         // of four accumulator quads each: dK and dV of a 16-feature tile
    constexpr int kWaveBytes = kTiles * 4 * 1024;      // [feature tile][dK, dV][16-key tile][lane][4 floats]
    const uint32_t lane_off = 16 * lane_now();
    unsigned char* const sums = reinterpret_cast<unsigned char*>(p.split_sums) + ((int64_t)bh * p.split_items + rank) * (4 * kWaveBytes) +
                                wave * kWaveBytes;
    static_for<kTiles>([&](auto tc) S2_INLINE {
      constexpr int ft = decltype(tc)::value;
      store_agent<0>(sums + 4096 * ft, lane_off, acc_dk[ft][0]);
      store_agent<1024>(sums + 4096 * ft, lane_off, acc_dk[ft][1]);
      store_agent<2048>(sums + 4096 * ft, lane_off, acc_dv[ft][0]);
      store_agent<3072>(sums + 4096 * ft, lane_off, acc_dv[ft][1]);
    });
    wait_all_loads();  // my stores have arrived
    __syncthreads();
    int* const flag = reinterpret_cast<int*>(&sm.rs[0]);
    if (wave == 0 && lane_off == 0) {
      int32_t* const count = p.split_count + (int64_t)bh * T + nth;
      *flag = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (*flag != parts - 1) return;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) acc_dk[ft][nt] = acc_dv[ft][nt] = f32x4{};
    const unsigned char* from = sums - (int64_t)part * (4 * kWaveBytes);
#pragma unroll 1
    for (int i = 0; i < parts; ++i, from += 4 * kWaveBytes) {
      static_for<kTiles / 4>([&](auto jc) S2_INLINE {
        constexpr int j = decltype(jc)::value;
        f32x4 x[16];
        load_agent16(from + 16384 * j, lane_off, x);
#pragma unroll
        for (int n = 0; n < 16; ++n) {
          f32x4& a = n & 2 ? acc_dv[4 * j + (n >> 2)][n & 1] : acc_dk[4 * j + (n >> 2)][n & 1];
          a += x[n];
        }
      });
    }
  }
  if (!wave_active) return;
  // dK and dV go out through LDS (free since the loop's last barrier; each wavefront uses regions of its
  // own, so no barrier).  A lane holds its row's features four at a time, and storing them from there
  // touches 32 rows per instruction with 16 bytes each; read back 16 bytes per lane, row after row, an
  // instruction stores four whole rows.
  constexpr int RS = D + 8;  // staging row stride (elements)
  const int ln_out = lane_now();
  static_assert(4 * 32 * (D + 8) <= 2 * Tile::kElems, "the staging rows fit two stages");
  uint16_t* sk_ = &sm.q[0][0] + wave * 32 * RS;
  uint16_t* sv_ = &sm.g[0][0] + wave * 32 * RS;
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      bf16x4 wk, wv;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        wk[e] = (__bf16)(acc_dk[ft][nt][e] * p.scale);
        wv[e] = (__bf16)(acc_dv[ft][nt][e]);
      }
      const int at = (16 * nt + (ln_out & 15)) * RS + 16 * ft + 4 * (ln_out >> 4);
      *reinterpret_cast<bf16x4*>(sk_ + at) = wk;
      *reinterpret_cast<bf16x4*>(sv_ + at) = wv;
    }
  uint16_t* dk_base = p.dk + kv_off;
  uint16_t* dv_base = p.dv + kv_off;
  constexpr int PPR = D / 8, RPI = 64 / PPR;  // 16-byte pieces per row, rows per instruction
#pragma unroll
  for (int i = 0; i < 32 / RPI; ++i) {
    const int r = RPI * i + ln_out / PPR, piece = ln_out % PPR;
    const u32x4 xk = *reinterpret_cast<const u32x4*>(sk_ + r * RS + 8 * piece);
    const u32x4 xv = *reinterpret_cast<const u32x4*>(sv_ + r * RS + 8 * piece);
    const int kr = key_of(r);
    if ((FINE || VARLEN) && kr >= N) continue;
    const int64_t o = (int64_t)kr * p.kv_st + 8 * piece;
    *reinterpret_cast<u32x4*>(dk_base + o) = xk;
    *reinterpret_cast<u32x4*>(dv_base + o) = xv;
  }
}

}  // namespace s2
