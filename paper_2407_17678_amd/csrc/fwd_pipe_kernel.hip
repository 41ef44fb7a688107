// Forward kernel: block-sparse causal attention with per-head lists of kept KV blocks (section 3.2:
// iterate K/V tiles of the kept blocks through on-chip memory, softmax over the kept keys only;
// section 4.2: which blocks a head keeps).  One workgroup owns a query tile of 128 rows that spans
// several mask rows (the Merge-Q idea of section 3.2: a big tile, a fine mask); it walks the merged
// list of KV blocks any of its rows keeps, 64 keys a step, and each of its four wavefronts (32 query
// rows) leaves out what its own mask rows do not keep.
//
// Orientation: the score tile is computed transposed, S^T = K Q^T, so that a lane owns one query (one
// column of the C layout).  Row max / row sum are then in-lane reductions plus one exchange with the
// other half of the wavefront, and the probabilities feed the second contraction O^T += V^T P^T
// straight from the accumulator registers.
//
// K and V chunks (64 keys) are brought in by direct global -> LDS loads, double buffered, each
// wavefront fetching 16 of the 64 rows (PieceTile in device_util.h); K is read as row fragments, V
// through the LDS transpose read.  The inner loop:
//
//   * it is software pipelined by one step: while the matrix pipe computes the scores of step i+1
//     and then P(i) V(i), the vector pipe turns the scores of step i into probabilities and finds
//     the maximum of step i+1;
//   * the interleave is written out by hand, one MFMA per slot with its share of the vector work,
//     LDS reads and direct loads, and fenced so that the compiler keeps it.  Measured on gfx950, a
//     SIMD only overlaps matrix and vector instructions that alternate finely in the instruction
//     streams; two wavefronts per SIMD then hide each other's scalar work and waits;
//   * the running maximum is only moved when a new score exceeds it, which after a few steps is rare: the
//     accumulators are rescaled in a branch.  Whole 128-row tiles of head_dim 128 and blocks of 64 or 128
//     tokens move it only when a score exceeds it by more than 2^kTau.  Everything else keeps it exact: a
//     row's largest probability is then 1, which rounding to bf16 leaves alone, and O of short rows is
//     closer to the exact result (relative error of O against 64 bits, exact and lazy: 2 x 4 heads x 4096 x
//     64, blocks of 64 2.10e-3 and 2.20e-3; 8192 x 128, blocks of 16 2.12e-3 and 2.25e-3);
//   * the direct loads of a tile are issued two or three to a write of M0 (their LDS targets are told
//     apart by the instruction's immediate offset);
//   * what a step needs to know (its first key, whether it is mine, where its rows lie) is formed inside the slots of the step
//     before it, without branches, and the fragment ring and the barrier lie there too: a scalar instruction is hidden
//     beside an MFMA, but takes a wavefront that has nothing else to do 10 cycles (its first use of a lane's value 30, a
//     compare and branch on vector values 38, a taken branch 22), and each step began with 75 of them.
//
// Before the last point and now (with a tile's start in tile_map.h), us, caches cold: 1 x 32 heads x 32768 x 128 1064 -> 1028, 4 x 16 x 8192 255 -> 246, 2 x 16 x 3904
// 52.1 -> 50.2, 2 x 16 x 4096 x 64 32.9 -> 30.6, 1 x 32 x 131072 in blocks of 128 6092 -> 5921, dense 1 x 32 x 8192 513 -> 508; with few tiles on the chip 1 x 4 x 512 x 64
// 9.8 -> 7.9, 128 rows x 32 heads against 30720 keys 50.8 -> 48.1.  (Direct loads one or two steps further ahead, in the LDS that a lone workgroup could have, change nothing there.)
//
// One loop serves both head sizes, blocks of 64 and 128 tokens and ragged ends (blocks of 16 and 32:
// fwd_gather_kernel.hip).  Against the phase-by-phase kernel that head_dim 64 and partial 128-row tiles used to
// run (per launch): 2 x 16 heads x 4096 x 64, blocks of 64: 38.3 -> 36.0 us; 2 x 16 x 3904 x 128 (61 blocks): 53.7 -> 48.8 us; a
// packed batch of 8 sequences of 200 to 8192 rows x 32 heads: 367 us in two launches -> 348 us in one.  What bounds it: with
// many steps per tile the matrix and vector pipes (head_dim 128 about 1.05 PFLOP/s; at 64 the vector work per MFMA
// doubles), with few the latency of a tile's start and end (10.8 us of a workgroup slot against 1.7 us per step; 7.8 and 1.7 at 64).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "config.h"
#include "device_util.h"
#include "kernels.h"
#include "sched_util.h"

namespace s2 {

namespace {

constexpr float kNegInf = -__builtin_inff();
constexpr unsigned kComputeUnits = 256;
constexpr float kTau = 8.0f;  // log2 units a score may exceed a lazily moved reference maximum by

// VARLEN: a packed batch of sequences of different lengths.  A workgroup finds its sequence's rows in
// cu_seqlens and treats them as a sequence of its own.  In its last, partial tile no lane fetches past
// the sequence's last token (keys after it lie after every query, which the causal mask drops) and
// stores are guarded per row.
template <int D, bool DENSE, bool VARLEN, bool LONE>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 3) void fwd_pipe_kernel(const AttnParams p) {
  typedef DmaTile<D> Tile;
  typedef PieceTile<D> Piece;
  __shared__ __attribute__((aligned(16))) uint16_t tiles[4][Tile::kElems];  // two stages of K, two of V
  uint16_t (*const sk)[Tile::kElems] = tiles, (*const sv)[Tile::kElems] = tiles + 2;
  constexpr int BM = kFwdBM, MW = 32, CH = 64;
  constexpr int KK = D / 16, DT = D / 32;
  constexpr int RB = Tile::kStride * 2;  // bytes per tile row
  constexpr int NQK = 2 * KK;  // MFMAs of the score contraction per step
  constexpr int NPV = 4 * DT;  // MFMAs of the second contraction per step
  constexpr int NS = NQK + NPV;
  constexpr int NG = Piece::kGroups;
  // LDS fragments are requested kLead MFMAs ahead (3 to 7 measure the same at D = 128; at D = 64 three keep a
  // wavefront at 168 registers, so that three fit a SIMD)
  constexpr int kLead = D == 128 ? 5 : 3, kRing = D == 64 ? kLead + 1 : 8;
  // The ring goes on from one step to the next, and across the barrier between them: it lies kLead slots before a step's end, when every
  // wavefront has asked for its last fragments.  (In packed batches at D = 64 it begins again with each step: no registers are left for
  // it, a Q fragment would be spilled.)
  // LONE: a run of rows against a cache, with a workgroup to a compute unit at most.  Its K and V come from HBM, one step ahead, and the ring's
  // early barrier only lengthens the wait for them: 4 x 8 heads, 768 rows against 44928 keys, 3 local + stride 11 (192 tiles) 84.6 us with
  // the ring going on, 76.5 with a new one each step; 2 x 27 heads, 128 rows against 45568 73.3 and 66.9; 1 x 32 heads x 64, 512 rows against 30720 42.2 and
  // 41.1.  (Two to a compute unit wait for each other's: 2048 rows against 44928 146.0 and 147.0.  A whole short sequence finds its keys in an L2: 1 x 8
  // x 2048 14.1 and 14.5.)
  constexpr bool kAcross = !LONE && (!VARLEN || D == 128);
  static_assert(!kAcross || (NS % kRing == 0 && kRing > kLead), "a fragment has the same place in every step");
  static_assert(!kAcross || 2 * NG <= NS - kLead, "all direct loads of a step are issued before its barrier");
  static_assert(!(DENSE && VARLEN), "the dense form walks 64-key blocks of whole sequences");

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int T = p.q_tiles.tiles_per_head;      // tiles of the whole sequence (indexes the lists)
  const int T_run = (p.q_rows + BM - 1) / BM;    // tiles this launch computes
  int bh, rank;
  if (!map_workgroup(p.row_map, blockIdx.x, bh, rank)) return;
  const int b = bh / p.by_heads, h = bh - b * p.heads;
  // longest tiles first: by the layout's order for a whole sequence, else simply last row first
  const bool whole = !VARLEN && p.q_row0 == 0 && T_run == T;
  int tile = p.q_row0 / BM + (T_run - 1 - rank), ent_lo = 0, n_ent = 0;
  if (!DENSE && whole) {
    const DevTiles::RowRec rec = p.q_tiles.row_rec(h, rank);
    tile = rec.tile;
    ent_lo = rec.ent_lo;
    n_ent = rec.n_ent;
  }
  // my sequence's length, its query rows in this call, and the rows of the tensors before it
  int N = p.seqlen, n_q = p.q_rows, row_base = 0;
  if (VARLEN) {
    const int lo = load_const<int32_t>(p.cu_seqlens + b), hi = load_const<int32_t>(p.cu_seqlens + b + 1);
    row_base = min(max(lo, 0), p.seqlen);  // whatever the array holds, stay inside the tensors
    N = min(min(max(hi - lo, 0), p.q_rows), p.seqlen - row_base);
    n_q = N;
    const int T_seq = (N + BM - 1) / BM;
    if (rank >= T_seq) return;
    tile = T_seq - 1 - rank;
  }
  const int S = DENSE ? CH : p.block_size;  // 64 or 128
  const int cpb_sh = S == 128 ? 1 : 0, cpb_m = (1 << cpb_sh) - 1, s_sh = 6 + cpb_sh;  // chunks per list entry; S as a shift
  const int qw0 = tile * BM + wave * MW;    // first query row of this wavefront (sequence position)
  const int ql0 = qw0 - p.q_row0;           // the same as a row of q / o / lse
  const bool wave_on = ql0 < n_q;           // whether I have query rows at all
  const int my_member = (wave * MW) >> s_sh;

  const int64_t q_off = (VARLEN ? row_base * p.q_st : b * p.q_sb) + h * p.q_sh;
  const int64_t kv_off = (VARLEN ? row_base * p.kv_st : b * p.kv_sb) + h * p.kv_sh;
  // minus the bias the grouped direct loads put into their lane offsets
  const char* kb = reinterpret_cast<const char*>(p.k + kv_off) - Piece::kBias;
  const char* vb = reinterpret_cast<const char*>(p.v + kv_off) - Piece::kBias;

  if (DENSE) {
    n_ent = min(N, (tile + 1) * BM) / CH;
  } else if (!whole) {
    ent_lo = load_const<int32_t>(p.q_tiles.ptr + h * T + tile);
    n_ent = load_const<int32_t>(p.q_tiles.ptr + h * T + tile + 1) - ent_lo;
  }
  const int total = n_ent << cpb_sh;  // steps: chunks of the entries
  if (total <= 0) return;
  EntryList list;
  if (!DENSE) list.init(p.q_tiles.ent + ent_lo, n_ent, lane);

  // Q^T fragments stay in registers for the whole tile (B operands of the score MFMAs); a lane without
  // a row of its own reads the last row, its result is never stored
  bf16x8 qf[KK];
  const int q_lane = min(ql0 + l32, n_q - 1);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    qf[kk] = *reinterpret_cast<const bf16x8*>(p.q + q_off + (int64_t)q_lane * p.q_st + 16 * kk + 8 * half);

  // Step j of the tile's list: its first key (0 past the end of a list, where entries are 0), and whether I have anything to
  // compute there: my mask rows keep some of it, and not every key lies after every one of my queries (q_end: past my last
  // one, 0 where I have none).
  const int q_end = wave_on ? qw0 + MW : 0;
  auto chunk_at = [&](int j, int& kv0, bool& act) S2_INLINE {
    if (DENSE) {
      kv0 = j * CH;
      act = kv0 < q_end;
    } else {
      const uint32_t e = (uint32_t)list.at(j >> cpb_sh);
      kv0 = (int)(e >> 16 << s_sh) + ((j & cpb_m) << 6);
      act = ((e >> my_member) & (uint32_t)(kv0 < q_end)) != 0;
    }
  };
  // how far (bytes) from the first key of my sequence the 16 rows lie that I fetch of the chunk that begins at key kv0
  const uint32_t row_bytes = (uint32_t)(2 * p.kv_st);  // (api.hip: at most 2^25)
  auto piece_row = [&](int kv0) S2_INLINE {
    if (DENSE) kv0 = min(kv0, (total - 1) * CH);
    return VARLEN ? min(kv0 + 16 * wave, N - 1) : kv0 + 16 * wave;
  };
  auto piece_off = [&](int row) S2_INLINE { return (uint64_t)(uint32_t)row * row_bytes; };

  f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = f32x16{};
  float m_ref = kNegInf;  // reference maximum (raw scores) of my query
  float mc = 0.f;         // the same times scale * log2(e); 0 while nothing was seen
  float l_run = 0.f;      // sum of the probabilities over my half's key rows
  const float c = p.scale_log2e;
  // how far a score may exceed the reference maximum before it is moved (raw scores; see the top of this file).  Finite, also
  // where 2^kTau is out of reach of any score: the first maximum has to move it from -inf.
  const bool lazy_ref = D == 128 && (VARLEN ? (tile + 1) * BM <= N : p.q_rows % BM == 0);
  const float tau = lazy_ref ? __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, fminf(kTau / c, 3.4e38f)))) : 0.f;
  // The lane offsets of my direct loads.  Where a packed sequence ends inside the 16 rows I fetch (VARLEN) no lane's goes past
  // end_off, the last piece of the last row that exists.
  const typename Piece::Plan plan = Piece::plan(p.kv_st, lane);
  auto end_off = [&](int row) S2_INLINE {
    return VARLEN && row + 16 > N ? (uint32_t)(N - 1 - row) * row_bytes + (2 * D - 16 + Piece::kBias) : ~0u;
  };
  // group g of the loads of my 16 rows, which start `off` bytes after the first key
  auto dma = [&](auto gc, const char* base, uint64_t off, uint32_t end, const uint16_t* stage) S2_INLINE {
    if constexpr (VARLEN) {
      typename Piece::Plan pl = plan;
#pragma unroll
      for (int n = 0; n < Piece::kLoads; ++n) pl.goff[n] = min(pl.goff[n], end - Piece::imm(n));
      Piece::template issue<decltype(gc)::value>(pl, base + off, stage, wave);
    } else {
      Piece::template issue<decltype(gc)::value>(plan, base + off, stage, wave);
    }
  };
  // lane parts of the addresses the fragments are read at
  const uint32_t k_lane = lds_addr(tiles) + l32 * RB + 16 * half, v_lane = lds_addr(tiles) + 2 * Tile::tr_base(lane);

  // scores [parity of the step][32-key half].  Zero to begin with: the registers of a step this
  // wavefront skips are still run through the exponential (with a shift of -inf) when the next step
  // is its own, so they must not hold a NaN; after a step they hold its probabilities.
  f32x16 s[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i >> 1][i & 1] = f32x16{};

  // ------------------------------------------------------------------ pieces of a step
  // The A operands of a step's MFMAs (head_dim 128: 16 row fragments of K, then 16 transposed fragments
  // of V; half as many at 64) pass through one ring of kRing registers sets, each requested from LDS kLead slots before
  // the MFMA that uses it.
  // fragment f: K fragment (kk = f / 2, key half f % 2) for f < NQK, else V^T fragment f - NQK
  // (group (f - NQK) / DT = key half, 16-key slab; feature tile (f - NQK) % DT)
  auto frag_load = [&](int f, uint32_t ks, uint32_t vs, bf16x8 (&fr)[kRing]) S2_INLINE {
    if (f < NQK)
      fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read16(ks, 32 * (f & 1) * RB + 32 * (f >> 1)));
    else
      fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read_tr(vs, 16 * ((f - NQK) / DT) * RB + 64 * ((f - NQK) % DT), RB));
  };
  // MFMA n of the score contraction of a step: kk = n / 2, key half = n % 2; fragment n
  auto qk_mfma = [&](int n, f32x16 (&sn)[2], const bf16x8 (&fr)[kRing]) S2_INLINE {
    const int kk = n >> 1, kt = n & 1;
    sn[kt] = mfma32(fr[n % kRing], qf[kk], kk == 0 ? f32x16{} : sn[kt]);
  };
  // MFMA n of the second contraction: group g = n / DT (key half g / 2, 16-key slab g % 2),
  // feature tile n % DT; fragment NQK + n
  auto pv_mfma = [&](int n, const bf16x8 (&fr)[kRing], const u32x4 (&pb)[4]) S2_INLINE {
    acc[n % DT] = mfma32(fr[(NQK + n) % kRing], __builtin_bit_cast(bf16x8, pb[n / DT]), acc[n % DT]);
  };
  // The probabilities of a step are made in three stages - scale and shift, exponential, sum and
  // pack - that a slot applies to different elements, so that no instruction waits for the one
  // before it.  Elements are numbered in the order the second contraction uses them:
  // e = 8 * g + i is score register 8 * (g % 2) + i of key half g / 2.  Stages 1 and 2 work in
  // place, in the score registers.
  auto p_stage1 = [&](int e0, int e1, f32x16 (&sc)[2]) S2_INLINE {
#pragma unroll
    for (int e = max(e0, 0); e < min(e1, 32); ++e) {
      const int g = e >> 3, r = 8 * (g & 1) + (e & 7);
      sc[g >> 1][r] = __builtin_fmaf(sc[g >> 1][r], c, -mc);
    }
  };
  auto p_stage2 = [&](int e0, int e1, f32x16 (&sc)[2]) S2_INLINE {
#pragma unroll
    for (int e = max(e0, 0); e < min(e1, 32); ++e) {
      const int g = e >> 3, r = 8 * (g & 1) + (e & 7);
      sc[g >> 1][r] = fast_exp2(sc[g >> 1][r]);
    }
  };
  auto p_stage3 = [&](int e0, int e1, f32x16 (&sc)[2], u32x4 (&pb)[4]) S2_INLINE {
#pragma unroll
    for (int e = max(e0, 0); e < min(e1, 32); ++e) {
      const int g = e >> 3, i = e & 7, r = 8 * (g & 1) + i;
      // the sum takes the unrounded probabilities: LSE is held to 1e-3, which a sum of bf16 values
      // cannot promise for rows with one or two keys
      l_run += sc[g >> 1][r];
      if (i & 1) {
        pb[g][i >> 1] = pack2(sc[g >> 1][r - 1], sc[g >> 1][r]);
      }
    }
  };
  // element index reached after slot sl: five elements every four slots, or (D = 64) three a slot
  constexpr int kPace = D == 128 ? 40 : 48;
  auto p_upto = [](int sl) S2_INLINE { return (kPace * (sl + 1)) / NS; };
  // drops what my query does not see of the step that begins at key kv0: keys after it
  auto mask_step = [&](f32x16 (&sn)[2], int kv0) S2_INLINE {
    const int ln = lane_now();  // (formed anew: at D = 64 no register is left for what the lane number gives)
#pragma unroll
    for (int pc = 0; pc < 4; ++pc) {
      const int row = kv0 + 16 * pc;
      // how many of these 16 keys I see, counted from the first one my half of the wavefront holds
      const int lim = qw0 + (ln & 31) - row + 1 - 4 * (ln >> 5);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (8 * (i >> 2) + (i & 3) >= lim) sn[pc >> 1][8 * (pc & 1) + i] = kNegInf;
    }
  };
  // running maximum over score registers r0 .. r1-1 (of 32)
  auto max_part = [&](int r0, int r1, const f32x16 (&sn)[2], float& mx) S2_INLINE {
#pragma unroll
    for (int r = r0; r < r1; r += 2) mx = fmaxf(fmaxf(mx, sn[r >> 4][r & 15]), sn[r >> 4][(r + 1) & 15]);
  };
  // moves the reference maximum where the new scores exceed it by more than tau (always for the first
  // step, when it is -inf) and rescales what has been accumulated so far
  auto update_ref = [&](float mx) S2_INLINE {
    // (a lane that has seen no key yet has m_ref = -inf: its first score always exceeds that, and while it
    // sees none the difference is not a number, which does not)
    if (__any(mx - m_ref > tau)) {
      const float m_new = fmaxf(m_ref, mx);
      const float m_use = (m_new == kNegInf) ? 0.f : m_new;
      const float alpha = fast_exp2((m_ref - m_use) * c);
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] *= alpha;
      m_ref = m_new;
      mc = m_use * c;
    }
  };
  // maximum of the scores in sn (masked on the diagonal), then the reference maximum; kv0: the step's first key
  auto finish_scores = [&](f32x16 (&sn)[2], int kv0, int act, float mx) S2_INLINE {
    if (kv0 + CH - 1 > qw0) {
      S2_FENCE();
      mask_step(sn, kv0);
      mx = kNegInf;
      max_part(0, 32, sn, mx);
      mx = max_halves(mx);
    }
    if (!act) mx = kNegInf;
    update_ref(mx);
  };

  // ------------------------------------------------------------------ prologue
  // A step this wavefront has nothing to compute in (its mask row drops the block, or every key
  // lies after its queries) runs through the same instruction stream when the step before or
  // after it is its own (see `step`); two such steps in a row are skipped.
  bool act_c, act_n;
  int kv_n;         // first key of the next step
  uint64_t off_n;   // where the key rows lie that I fetch of it, and where they end
  uint32_t end_n;
  {
    int kv_c;
    chunk_at(0, kv_c, act_c);
    chunk_at(1, kv_n, act_n);
    const int row_c = piece_row(kv_c), row_n = piece_row(kv_n);
    const uint64_t off_c = piece_off(row_c);
    const uint32_t end_c = end_off(row_c);
    off_n = piece_off(row_n);
    end_n = end_off(row_n);
    static_for<NG>([&](auto gc) S2_INLINE {
      dma(gc, kb, off_c, end_c, sk[0]);
      dma(gc, vb, off_c, end_c, sv[0]);
    });
    static_for<NG>([&](auto gc) S2_INLINE { dma(gc, kb, off_n, end_n, sk[1]); });
  }
  wait_all_loads();
  __syncthreads();
  if (act_c) {
    bf16x8 fr[kRing];
#pragma unroll
    for (int f = 0; f < kLead; ++f) frag_load(f, k_lane, 0, fr);
    static_for<NQK>([&](auto nc) S2_INLINE {
      constexpr int n = decltype(nc)::value;
      if constexpr (n + kLead < NQK) frag_load(n + kLead, k_lane, 0, fr);
      qk_mfma(n, s[0], fr);
      S2_FENCE();
    });
  }
  {
    int kv_c;
    chunk_at(0, kv_c, act_c);
    float mx = kNegInf;
    if (kv_c + CH - 1 <= qw0) {
      max_part(0, 32, s[0], mx);
      mx = max_halves(mx);
    }
    finish_scores(s[0], kv_c, act_c, mx);
  }
  __syncthreads();  // all wavefronts are done with K(0) before step 0 loads K(2) over it

  // ------------------------------------------------------------------ one step
  // While step `it` runs, K(it+1) and V(it) are in LDS, sc holds the scores of step it and the reference
  // maximum already covers them.
  int it = 0;
  int kv_nn;           // the step after the next one
  bool act_nn;
  uint64_t off_nn;
  uint32_t end_nn;
  uint32_t ks, vs;     // where the lane's fragments of this step's K and V are
  bf16x8 fr[kRing];
  // what step `it` (of parity par) needs to know
  auto open_step = [&](auto pc) S2_INLINE {
    constexpr int par = decltype(pc)::value;
    chunk_at(it + 2, kv_nn, act_nn);
    const int row_nn = piece_row(kv_nn);
    off_nn = piece_off(row_nn);
    end_nn = end_off(row_nn);
    // Where one of the two steps is not mine its scores stay out of the maximum and its probabilities are 0,
    // and the rows of the other one stand in for its own: whatever the rows hold that I do not attend, the scores
    // are finite (so that the probabilities are 0) and nothing of them is accumulated.
    ks = k_lane + (uint32_t)Tile::kBytes * (act_n ? par ^ 1 : 2 + par);
    vs = v_lane + (uint32_t)Tile::kBytes * (act_c ? 2 + par : par ^ 1);
    asm volatile("" : "+v"(ks), "+v"(vs));
  };
  // From step `it` to the next: everything this one loads has landed, and every wavefront has read what it needs of it
  auto next_step = [&](auto pc) S2_INLINE {
    constexpr int par = decltype(pc)::value;
    wait_all_loads();
    __syncthreads();
    it = __builtin_amdgcn_readfirstlane(it + 1);
    act_c = act_n;
    off_n = off_nn;
    end_n = end_nn;
    kv_n = kv_nn;
    act_n = act_nn;
    open_step(std::integral_constant<int, par ^ 1>{});
  };
  auto first_frags = [&]() S2_INLINE {
#pragma unroll
    for (int f = 0; f < kLead; ++f) frag_load(f, ks, vs, fr);
  };
  auto step = [&](auto pc, f32x16 (&sc)[2], f32x16 (&sn)[2]) S2_INLINE {
    constexpr int par = decltype(pc)::value;
    // group d of this step's direct loads: 0..NG-1 for K(it+2), into the stage K(it) was in, then
    // V(it+1), into the stage V(it-1) was in
    auto step_dma = [&](auto dc) S2_INLINE {
      constexpr int d = decltype(dc)::value;
      if constexpr (d < NG)
        dma(dc, kb, off_nn, end_nn, sk[par]);
      else
        dma(std::integral_constant<int, d - NG>{}, vb, off_n, end_n, sv[par ^ 1]);
    };
    // keeps the entry window moving, two steps at a time: what is asked for until the next time is of steps it + 3 and it + 4
    if (!DENSE && par == 0) (void)list.get((it + 2) >> cpb_sh, lane_now());
    if (act_c || act_n) {
      // a step that is not mine: every probability exp2(s*c - inf) = 0
      const float mc_keep = mc;
      if (!act_c) mc = __builtin_inff();
      const int kv_s = __builtin_amdgcn_readfirstlane(kv_n);
      const bool act_s = act_n;
      u32x4 pb[4];
      float mx = kNegInf;
      if constexpr (!kAcross) first_frags();
      S2_FENCE();
      // NQK + NPV slots, one MFMA each
      static_for<NS>([&](auto slc) S2_INLINE {
        constexpr int sl = decltype(slc)::value;
        if constexpr (kAcross && sl + kLead == NS) next_step(pc);
        if constexpr (kAcross || sl + kLead < NS) frag_load((sl + kLead) % NS, ks, vs, fr);
        if constexpr (sl < NQK)
          qk_mfma(sl, sn, fr);
        else
          pv_mfma(sl - NQK, fr, pb);
        // probabilities of this step, each stage one slot behind the one before it (elements
        // 8 g .. 8 g + 7 are packed before slot NQK + DT * g, where their MFMAs start)
        static_assert(kPace * (NQK - 2) / NS >= 8 && kPace * (NQK + 3 * DT - 2) / NS >= 32, "packed in time");
        p_stage1(p_upto(sl - 1), p_upto(sl), sc);
        p_stage2(p_upto(sl - 2), p_upto(sl - 1), sc);
        p_stage3(p_upto(sl - 3), p_upto(sl - 2), sc, pb);
        // maximum of the next step's scores, once its MFMAs are done
        constexpr int kMaxSlots = D == 128 ? 8 : 6, kMaxStep = D == 128 ? 4 : 6;
        static_assert(NQK + 1 + kMaxSlots <= NS - 1 && kMaxSlots * kMaxStep >= 32, "all 32 registers");
        if constexpr (sl >= NQK + 2 && sl < NQK + 2 + kMaxSlots)
          max_part(kMaxStep * (sl - NQK - 2), std::min(32, kMaxStep * (sl - NQK - 1)), sn, mx);
        if constexpr (sl == std::min(NS - 1, NQK + 2 + kMaxSlots)) mx = max_halves(mx);
        // Nothing to execute: ties the running sum and maximum to this slot, or the optimiser
        // collects their additions and comparisons after the last MFMA.
        asm volatile("" : "+v"(l_run), "+v"(mx));
        if constexpr (sl < 2 * NG) step_dma(std::integral_constant<int, sl>{});
        S2_FENCE();
      });
      mc = mc_keep;
      finish_scores(sn, kv_s, act_s, mx);
      if constexpr (!kAcross) next_step(pc);
    } else {
      static_for<2 * NG>([&](auto dc) S2_INLINE { step_dma(dc); });
      next_step(pc);
      if constexpr (kAcross) first_frags();
    }
  };

  constexpr std::integral_constant<int, 0> even;
  constexpr std::integral_constant<int, 1> odd;
  open_step(even);
  if constexpr (kAcross) first_frags();
  // (after the last step the wavefronts still have fragments on their way, from inside the stages, that nothing uses)
  for (;;) {
    step(even, s[0], s[1]);
    if (it >= total) break;
    step(odd, s[1], s[0]);
    if (it >= total) break;
  }

  // ------------------------------------------------------------------ epilogue
  if (!wave_on) return;
  const float l_tot = sum_halves(l_run);
  store_rows<D, VARLEN>(acc, 1.0f / l_tot, sk[0] + wave * MW * (D + 8), p.o + q_off + (int64_t)ql0 * p.q_st, p.q_st, n_q - ql0, lane);
  const int64_t lse_row = VARLEN ? (int64_t)h * p.seqlen + row_base + ql0 + l32  // [heads, rows of the tensors]
                                 : ((int64_t)b * p.heads + h) * p.q_rows + ql0 + l32;
  if (half == 0 && (!VARLEN || ql0 + l32 < n_q)) p.lse[lse_row] = m_ref * p.scale + __logf(l_tot);
}

template <int D>
hipError_t launch_one(const AttnParams& p, bool dense, hipStream_t stream) {
  const dim3 grid(p.row_map.grid()), block(kThreads);
  if (dense)
    hipLaunchKernelGGL((fwd_pipe_kernel<D, true, false, false>), grid, block, 0, stream, p);
  else if (p.cu_seqlens)
    hipLaunchKernelGGL((fwd_pipe_kernel<D, false, true, false>), grid, block, 0, stream, p);
  else if (p.q_rows < p.seqlen && grid.x <= kComputeUnits)
    hipLaunchKernelGGL((fwd_pipe_kernel<D, false, false, true>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((fwd_pipe_kernel<D, false, false, false>), grid, block, 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd(const AttnParams& params, bool dense, hipStream_t stream) {
  AttnParams p = params;
  const int pairs = p.batch * p.heads, tiles = (p.q_rows + kFwdBM - 1) / kFwdBM;
  p.row_map = row_map(pairs, tiles, map_group(pairs, tiles, p.cu_seqlens != nullptr), dense ? kDenseRows : p.q_rows < p.seqlen ? kRowsOfCache : kSparseRows,
                      xcd_slots(p.head_dim));
  p.by_heads = fast_div(p.heads);
  if (!dense && p.block_size < 64) return launch_fwd_gather(p, stream);
  return p.head_dim == 128 ? launch_one<128>(p, dense, stream) : launch_one<64>(p, dense, stream);
}

}  // namespace s2
