// One workgroup's share of the dQ launch: a tile of 128 query rows, the row-stationary half of the backward pass (the gradient of the forward of section 3.2).
// Same tiles, lists, staging and orientation as the forward (fwd_pipe_kernel.hip) - a workgroup owns 128
// query rows, a wavefront 32 of them, and walks the 64-key chunks of the KV blocks its mask rows keep,
// recomputing P and forming dS = P * (dP - delta), dQ += scale * dS K; where dK/dV is a later launch it also computes
// delta = rowsum(dO * O) and leaves the row statistics in the workspace for it - with a hand-scheduled inner loop:
//
//   * it runs in half chunks of 32 keys, skewed by one half: S and dP of the next half are computed
//     around the dQ MFMAs of this one, with this half's dS arithmetic under the former and the next
//     half's exponentials under the latter;
//   * the order is written out, one fragment and two 16x16x32 MFMAs per slot with their share of the vector work and LDS reads,
//     and fenced so that the compiler keeps it (see sched_util.h for the measurements
//     behind this); the A operands pass through a ring of registers requested a few slots ahead;
//   * the direct loads of a tile are issued two or three to a write of M0.
//
// Head_dim 64, mask blocks below 64 tokens (FINE: chunks gathered from 16-key pieces) and ragged ends
// (VARLEN) are the same loop, as in the forward.  Against the phase-by-phase kernel that these used to run,
// per launch: 2 x 16 heads x 4096 x 64, blocks of 64: 50.1 -> 45.9 us; 2 x 16 x 3904 x 128 (61 blocks):
// 73.3 -> 65.2 us; 1 x 16 x 8192 x 128, blocks of 16: 84.2 -> 70 us; a packed batch of 8 sequences of 200 to
// 8192 rows x 32 heads: 497 us in two launches -> 478 us in one.  It is bound as the forward is: by the
// matrix pipe and the vector work beside it over long lists, by a tile's start and end over short ones.  The 16x16x32 shape (less power
// to a flop and fewer bank conflicts, see dkdv_tile.h), dP's contraction beginning at -delta instead of a subtraction a pair, and no chunk
// fetched past a list's end, together: 1 x 32 x 32768 x 128 1.438 -> 1.385 ms, 4 x 32 x 8192 x 64 457 -> 425 us, 3 x 20 x 8192 x 64 with 32-token
// blocks 138 -> 129, 2 x 16 x 3904 x 128 61.0 -> 59.2.  (One rolled loop of half steps whose ring goes on across the barriers, as in dK/dV,
// was built: the same over long lists, 6 to 15 % slower over short ones, where its scalar work is not hidden.)
#pragma once
#include <hip/hip_runtime.h>

#include "config.h"
#include "device_util.h"
#include "kernels.h"
#include "sched_util.h"

namespace s2 {

constexpr float kDropped = -__builtin_inff();  // score of a pair that the mask drops

template <int D>
struct DqPipeSmem {
  uint16_t k[2][ChunkTile<D>::kElems];
  uint16_t v[2][ChunkTile<D>::kElems];
};

// STATS: the launch runs before dK/dV and leaves the row statistics for it; else they are there already.
template <int D, bool DENSE, bool FINE, bool VARLEN, bool STATS>
__device__ __forceinline__ void dq_tile(const AttnParams& p, int wg, unsigned char* smem_raw) {
  typedef ChunkTile<D> Tile;
  typedef PieceTile<D, Tile> Piece;
  DqPipeSmem<D>& sm = *reinterpret_cast<DqPipeSmem<D>*>(smem_raw);
  constexpr int BM = kBwdBM, MW = 32, CH = 64;
  constexpr int KS = D / 32, FT = D / 16;  // 32-feature steps of S and dP, 16-feature tiles of dQ
  constexpr int KK = D / 16;               // fragments of each contraction, two MFMAs each
  static_assert(2 * KS == KK && FT == KK, "two 16-key tiles by KS steps; one 32-key slab by FT tiles");
  constexpr int NG = Piece::kGroups;
  constexpr int RB = Tile::RB;             // bytes per tile row
  constexpr int kSlots = 3 * KK;           // fragments per half step: KK of S, KK of dQ, KK of dP
  constexpr int kLead = D == 128 ? 5 : 3, kRing = kLead + 1;
  static_assert(!(DENSE && (FINE || VARLEN)), "the dense form walks 64-key blocks of whole sequences");

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  if (STATS && !DENSE && !VARLEN) clear_split_counts(p, wg * kThreads + tid);
  const int T = p.q_tiles.tiles_per_head;
  int bh, rank;
  if (!map_workgroup(p.row_map, wg, bh, rank)) return;
  const int b = bh / p.by_heads, h = bh - b * p.heads;
  int tile = T - 1 - rank, ent_lo = 0, n_ent = 0;
  if (!DENSE && !VARLEN) {
    const DevTiles::RowRec rec = p.q_tiles.row_rec(h, rank);
    tile = rec.tile;
    ent_lo = rec.ent_lo;
    n_ent = rec.n_ent;
  }
  int N = p.seqlen, row_base = 0;  // my sequence's length, and the rows of the tensors before it
  if (VARLEN) {
    const int lo = load_const<int32_t>(p.cu_seqlens + b), hi = load_const<int32_t>(p.cu_seqlens + b + 1);
    row_base = min(max(lo, 0), p.seqlen);  // whatever the array holds, stay inside the tensors
    N = min(min(max(hi - lo, 0), p.q_rows), p.seqlen - row_base);
    const int T_seq = (N + BM - 1) / BM;
    if (rank >= T_seq) return;
    tile = T_seq - 1 - rank;
  }
  const int S = DENSE ? CH : p.block_size;  // FINE: 16 or 32, else 64 or 128
  const int cpb_sh = S == 128 ? 1 : 0, cpb_m = (1 << cpb_sh) - 1, s_sh = 6 + cpb_sh;  // chunks per list entry; S of one as a shift
  const int ppe_sh = S == 32 ? 1 : 0;                              // FINE: 16-key pieces per list entry
  const int qw0 = tile * BM + wave * MW;  // first query row of this wavefront
  const bool wave_on = qw0 < N;           // whether I have query rows at all
  const int my_member = (wave * MW) >> s_sh;  // (not FINE)

  const int64_t q_off = (VARLEN ? row_base * p.q_st : b * p.q_sb) + h * p.q_sh;
  const int64_t kv_off = (VARLEN ? row_base * p.kv_st : b * p.kv_sb) + h * p.kv_sh;
  // minus the bias the grouped direct loads put into their lane offsets
  const char* kb = reinterpret_cast<const char*>(p.k + kv_off) - Piece::kBias;
  const char* vb = reinterpret_cast<const char*>(p.v + kv_off) - Piece::kBias;
  const uint32_t row_bytes = (uint32_t)(2 * p.kv_st);  // (api.hip: at most 2^25)

  if (DENSE) {
    n_ent = min(N, (tile + 1) * BM) / CH;
  } else if (VARLEN) {
    ent_lo = load_const<int32_t>(p.q_tiles.ptr + h * T + tile);
    n_ent = load_const<int32_t>(p.q_tiles.ptr + h * T + tile + 1) - ent_lo;
  }
  // chunks: those of an entry, or (FINE) as many as the entries' pieces fill
  const int total = FINE ? ((n_ent << ppe_sh) + 3) >> 2 : n_ent << cpb_sh;
  if (total <= 0) return;
  EntryList list;
  if (!DENSE) list.init(p.q_tiles.ent + ent_lo, n_ent, lane);
  // FINE: piece pc (0..3) of chunk j: its first key row, and which of my two groups of 16 query rows keep
  // it (bits 0 and 1; both or neither for 32-token blocks)
  auto piece_at = [&](int j, int pc, int& row, int& bits) S2_INLINE {
    const int x = 4 * j + pc;
    const int i = x >> ppe_sh;
    const uint32_t e = (uint32_t)list.peek(min(i, n_ent - 1));
    row = (int)(e >> 16) * S + ((x & ppe_sh) << 4);
    bits = ppe_sh ? ((e >> wave) & 1) * 3 : (e >> (2 * wave)) & 3;
    if (i >= n_ent) bits = 0;
  };
  const uint32_t late_from = (uint32_t)(qw0 >> (4 + ppe_sh)) << 16;  // FINE: entries from my first row's block on
  const int q_end = wave_on ? qw0 + MW : 0;  // past my last query
  // Chunk j of the tile's list: the first key row of the 16 that I fetch (past the end any that exist), and
  // for either 32-key half whether I have anything to compute in it (bit kt: my mask rows keep some of
  // it and not every key lies after every one of my queries), whether some of it has to be masked
  // for me (bit 2 + kt) and (FINE) which of its pieces are mine (bits 4 + 2 * kt and 5 + 2 * kt).
  auto chunk_at = [&](int j, int& row, int& state) S2_INLINE {
    const bool inside = j < total;
    state = 0;
    if constexpr (FINE) {
      // every lane's entry at once (0 after the end of the list: kept by nobody), then the chunk's bits
      const int i0 = (4 * j) >> ppe_sh;
      const int src = (i0 >> 6) != list.batch ? list.nxt : list.cur;  // a chunk's entries are of one batch
      const uint32_t mine = (uint32_t)__builtin_amdgcn_readlane(src, (i0 + (wave >> ppe_sh)) & 63);
      row = (int)(mine >> 16) * S + ((wave & ppe_sh) << 4);
      const int bits = ppe_sh ? ((src >> wave) & 1) * 3 : (src >> (2 * wave)) & 3;
      const uint64_t any = __ballot(bits != 0), whole = __ballot(bits == 3) & ~__ballot((uint32_t)src >= late_from);
      int on = (int)(any >> (i0 & 63)) & 15, all = (int)(whole >> (i0 & 63)) & 15;
      if (ppe_sh) {  // two pieces to an entry
        on = ((on & 1) | ((on & 2) << 1)) * 3;
        all = ((all & 1) | ((all & 2) << 1)) * 3;
      }
      state = (on & 3 ? 1 : 0) | (on & 12 ? 2 : 0) | ((all & 3) != 3 ? 4 : 0) | ((all & 12) != 12 ? 8 : 0) | on << 4;
    } else {
      // (branches kept out: past a list's end entries are 0, kept by nobody, and dense chunks lie past q_end)
      int kv0, keep = 3;
      if (DENSE) {
        kv0 = j * CH;
        row = min(kv0, (total - 1) * CH) + 16 * wave;
      } else {
        const uint32_t e = (uint32_t)list.at(j >> cpb_sh);
        kv0 = (int)(e >> 16 << s_sh) + ((j & cpb_m) << 6);
        keep = 3 * ((e >> my_member) & 1);
        row = kv0 + 16 * wave;
      }
      const int seen = q_end - kv0;  // half kt: mine if more than 32 * kt, masked if less than 32 * kt + 63
      state = (keep & ((int)(seen > 0) | (int)(seen > 32) << 1)) | (int)(seen < 63) << 2 | (int)(seen < 95) << 3;
    }
    if (FINE && (!inside || !wave_on)) state &= ~3;
    if (VARLEN) row = min(row, N - 1);
  };

  // Q^T and dO^T fragments (B operands), lane % 16 = query; delta = rowsum(dO * O) of my query from the
  // dO fragments (8 features of every 32 in each of the four lane groups, added up with the lane 32 away and then with the one
  // 16 away: the order that delta_kernel keeps to, bit for bit), written out with LSE as the dK/dV kernel, which runs after
  // this one, wants them.  A lane without a row of its own reads the last row; nothing of it is stored.
  // [32-feature step][16-query tile nt]
  bf16x8 qf[KS][2], gf[KS][2];
  float delta_l[2], lse_l[2];
  bf16x8 of[KS][2];
  int64_t stat_row[2];
  // (all loads first, while the list is on its way: a wait between them would be a second trip to memory at every tile's start)
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int my_row = min(qw0 + 16 * nt + l16, N - 1);
    const int64_t at = q_off + (int64_t)my_row * p.q_st + 8 * g;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      qf[kk][nt] = *reinterpret_cast<const bf16x8*>(p.q + at + 32 * kk);
      gf[kk][nt] = *reinterpret_cast<const bf16x8*>(p.d_o + at + 32 * kk);
      if (STATS) of[kk][nt] = *reinterpret_cast<const bf16x8*>(p.o + at + 32 * kk);
    }
    stat_row[nt] = VARLEN ? (int64_t)h * p.seqlen + row_base + my_row  // [heads, rows of the tensors]
                          : ((int64_t)b * p.heads + h) * N + my_row;
    lse_l[nt] = p.lse[stat_row[nt]];
    if (!STATS) delta_l[nt] = -p.neg_delta[stat_row[nt]];
  }
  typename Piece::Plan plan = Piece::plan(p.kv_st, lane);
  auto issue_chunk = [&](int row, int stage) S2_INLINE {
    // where a packed sequence ends inside the rows I fetch they are limited to the rows that exist; the
    // lists ascend, so from then on every piece is such a piece, with fewer and fewer rows
    if (VARLEN && row + 16 > N) Piece::limit(plan, N - row, p.kv_st);
    const uint64_t at = (uint64_t)(uint32_t)row * row_bytes;
    const char *kg = kb + at, *vg = vb + at;
    static_for<NG>([&](auto gc) S2_INLINE {
      constexpr int n = decltype(gc)::value;
      Piece::template issue<n>(plan, kg, sm.k[stage], wave);
      Piece::template issue<n>(plan, vg, sm.v[stage], wave);
    });
  };
  int row_n, state_c, state_n;
  {
    int row_c;
    chunk_at(0, row_c, state_c);
    chunk_at(1, row_n, state_n);
    issue_chunk(row_c, 0);
  }

  S2_FENCE();
#pragma unroll
  for (int nt = 0; STATS && nt < 2; ++nt) {
    float part = 0.f;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int e = 0; e < 8; ++e) part = __builtin_fmaf((float)gf[kk][nt][e], (float)of[kk][nt][e], part);
    delta_l[nt] = sum_groups(part);
  }
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    if (STATS && g == 0 && qw0 + 16 * nt + l16 < N) {
      p.neg_delta[stat_row[nt]] = -delta_l[nt];
      p.neg_lse[stat_row[nt]] = lse_l[nt] * p.neg_inv_scale;
    }
    lse_l[nt] *= 1.4426950408889634f;
  }

  f32x4 acc[FT][2];  // dQ transposed [16-feature tile][16-query tile]: lane % 16 = query, register r = feature 4 * g + r
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) acc[ft][nt] = f32x4{};
  // what the dP contraction begins with, so that it ends at dP - delta (a subtraction less a pair)
  f32x4 dp0[2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) dp0[nt] = f32x4{-delta_l[nt], -delta_l[nt], -delta_l[nt], -delta_l[nt]};
  const float c = p.scale_log2e;
  // lane parts of the addresses the fragments are read at (stage 0 of K; V lies v_from_k further on)
  const uint32_t k_lane = lds_addr(sm.k[0]) + Tile::row_lane(lane), tr_lane = lds_addr(sm.k[0]) + Tile::tr_lane(lane);
  constexpr uint32_t v_from_k = sizeof(sm.k);

  // Scores of a 32-key half [16-key tile m][16-query tile nt]: register r is key 4 * g + r of the tile, lane % 16 the query.
  // sc holds S, then P in place; dp holds dP - delta, then dS in place.
  f32x4 sc[2][2][2], dp[2][2];  // sc[parity of the half]
  u32x4 dsb[2];                 // dS of this half as B operands [16-query tile]
  // element x (0..15), in the order of the B operands
#define S2_AT(a, x) (a)[((x) >> 2) & 1][(x) >> 3][(x) & 3]

  // Drops what my queries do not see of half kt of chunk j: keys after them and (FINE) pieces their mask row
  // does not keep.  (A half that is not mine at all gets lse = +inf instead: P = dS = 0.)
  auto mask_half = [&](f32x4 (&s2)[2][2], int j, int kt) S2_INLINE {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      int row, bits = 3;
      if constexpr (FINE) {
        piece_at(j, 2 * kt + m, row, bits);
      } else if (DENSE) {
        row = j * CH + 32 * kt + 16 * m;
      } else {
        row = (list.peek(j >> cpb_sh) >> 16) * S + (j & cpb_m) * CH + 32 * kt + 16 * m;
      }
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        if (FINE && !((bits >> nt) & 1)) {  // the mask row of these queries drops the piece
          s2[m][nt] = f32x4{kDropped, kDropped, kDropped, kDropped};
        } else if (row + 15 > qw0 + 16 * nt) {
          // how many of the piece's keys my query sees, counted from the first one that my lane holds
          const int lim = qw0 + 16 * nt + l16 - row + 1 - 4 * g;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (r >= lim) s2[m][nt][r] = kDropped;
        }
      }
    }
  };

  bool act_cur = false;  // whether the half whose P is in sc[parity] is mine
  int on_cur = 3;        // FINE: which of its pieces are

  // ------------------------------------------------------------------ prologue
  wait_all_loads();
  __syncthreads();
  // S, dP and P of the first half, one after the other
  {
    const uint32_t k_row = k_lane, v_row = k_lane + v_from_k;
#pragma unroll
    for (int f = 0; f < KK; ++f) {
      const int m = f & 1, kk = f >> 1;
      const bf16x8 kr = __builtin_bit_cast(bf16x8, lds_read16(k_row, Tile::row_off(m, kk))), vr = __builtin_bit_cast(bf16x8, lds_read16(v_row, Tile::row_off(m, kk)));
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        sc[0][m][nt] = mfma16(kr, qf[kk][nt], kk == 0 ? f32x4{} : sc[0][m][nt]);
        dp[m][nt] = mfma16(vr, gf[kk][nt], kk == 0 ? dp0[nt] : dp[m][nt]);
      }
    }
    act_cur = state_c & 1;
    on_cur = (state_c >> 4) & 3;
    if (state_c & 4) mask_half(sc[0], 0, 0);
#pragma unroll
    for (int x = 0; x < 16; ++x) S2_AT(sc[0], x) = fast_exp2(__builtin_fmaf(S2_AT(sc[0], x), c, act_cur ? -lse_l[x >> 3] : kDropped));
    if (!act_cur || (FINE && on_cur != 3)) {  // (what does not come from a piece of mine may not be a number)
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (!act_cur || !((on_cur >> ((x >> 2) & 1)) & 1)) S2_AT(sc[0], x) = S2_AT(dp, x) = 0.f;
    }
  }

  // ------------------------------------------------------------------ one half step
  // On entry: sc[PAR] holds P of this half (half KT of the chunk in stage stc), dp its dP; K / V of
  // the next half's chunk are in stage stn (the same stage for KT = 0).
  // jn, state_x: the next half's chunk and its state.
  auto half_step = [&](auto par_c, auto kt_c, int stc, int stn, int jn, int state_x) S2_INLINE {
    constexpr int PAR = decltype(par_c)::value, KT = decltype(kt_c)::value;
    constexpr int KTN = KT ^ 1;  // which half of its chunk the next half is
    const bool act_n = (state_x >> KTN) & 1, masked_n = (state_x >> (2 + KTN)) & 1;
    // Neither this half nor the next is mine (mask row drops them, or their keys lie after my
    // queries): nothing to compute; the next half's P and dP are zero.  One of the two being mine
    // runs the whole stream (the other's probabilities are zero through lse = +inf), with its rows standing in for
    // the other's: whatever the rows hold that I do not attend, S and dP are finite and dS exactly 0.  Likewise
    // (FINE) the piece that is mine for one of the same half that is not.
    const bool act_this = act_cur;
    const int on_this = on_cur, on_n = (state_x >> (4 + 2 * KTN)) & 3;
    act_cur = act_n;
    on_cur = on_n;
    if (!act_this && !act_n) {
#pragma unroll
      for (int x = 0; x < 16; ++x) S2_AT(sc[PAR ^ 1], x) = S2_AT(dp, x) = 0.f;
      return;
    }
    const uint32_t from_n = stn * (uint32_t)Tile::kBytes + 32 * KTN * RB, from_this = stc * (uint32_t)Tile::kBytes + 32 * KT * RB;
    const uint32_t row_off = act_n ? from_n : from_this, tr_off = act_this ? from_this : from_n;
    // rows of the next half's 16-key tiles, and of this half's (the transposed fragments hold both)
    uint32_t k_row = k_lane + row_off, k_row1 = k_row, k_tr = tr_lane + tr_off, k_tr1 = k_tr;
    if constexpr (FINE) {
      const int on_r = act_n ? on_n : on_this, on_t = act_this ? on_this : on_n;
      if (on_r == 2) k_row += 16 * RB;
      if (on_r == 1) k_row1 -= 16 * RB;
      if (on_t == 2) k_tr += 16 * RB;
      if (on_t == 1) k_tr1 -= 16 * RB;
    }
    asm volatile("" : "+v"(k_row), "+v"(k_tr));
    if constexpr (FINE) asm volatile("" : "+v"(k_row1), "+v"(k_tr1));
    bf16x8 fr[kRing];
    // fragment f of the half step, in the order the MFMAs use them: KK row fragments of the next half's K (tile f % 2, step f / 2), KK
    // transposed fragments of this half's K (feature tile), KK row fragments of the next half's V
    auto frag_load = [&](auto fc) S2_INLINE {
      constexpr int f = decltype(fc)::value;
      const uint32_t row_at = FINE && (f & 1) ? k_row1 : k_row;
      if constexpr (f < KK)
        fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read16(row_at, Tile::row_off(f & 1, f >> 1)));
      else if constexpr (f < 2 * KK)
        fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read_tr2(k_tr, FINE ? k_tr1 : k_tr, Tile::tr_off(0, f - KK), Tile::tr_off(0, f - KK) + 16 * RB));
      else
        fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read16(row_at, v_from_k + Tile::row_off(f & 1, (f - 2 * KK) >> 1)));
    };
    static_for<kLead>([&](auto fc) S2_INLINE { frag_load(fc); });
    float neg_ln[2] = {act_n ? -lse_l[0] : kDropped, act_n ? -lse_l[1] : kDropped};
    S2_FENCE();
    static_for<kSlots>([&](auto nc) S2_INLINE {
      constexpr int n = decltype(nc)::value;
      if constexpr (n + kLead < kSlots) frag_load(std::integral_constant<int, n + kLead>{});
      // the two MFMAs of the slot
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        if constexpr (n < KK) {  // S of the next half
          constexpr int m = n & 1, kk = n >> 1;
          sc[PAR ^ 1][m][nt] = mfma16(fr[n % kRing], qf[kk][nt], kk == 0 ? f32x4{} : sc[PAR ^ 1][m][nt]);
        } else if constexpr (n < 2 * KK) {  // dQ of this half: feature tile
          acc[n - KK][nt] = mfma16(fr[n % kRing], __builtin_bit_cast(bf16x8, dsb[nt]), acc[n - KK][nt]);
        } else {  // dP of the next half
          constexpr int m = n & 1, kk = (n - 2 * KK) >> 1;
          dp[m][nt] = mfma16(fr[n % kRing], gf[kk][nt], kk == 0 ? dp0[nt] : dp[m][nt]);
        }
      }
      // dS = P * (dP - delta) of this half under the S MFMAs, complete and packed before dQ begins
      constexpr int ND = KK - 1;
      auto dupto = [](int i) { return i >= ND ? 16 : (16 * i + ND - 1) / ND; };
      if constexpr (n < ND) {
#pragma unroll
        for (int x = dupto(n); x < dupto(n + 1); ++x) S2_AT(dp, x) *= S2_AT(sc[PAR], x);
      }
      if constexpr (n == KK - 1) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          dsb[nt] = u32x4{pack2(dp[0][nt][0], dp[0][nt][1]), pack2(dp[0][nt][2], dp[0][nt][3]), pack2(dp[1][nt][0], dp[1][nt][1]),
                          pack2(dp[1][nt][2], dp[1][nt][3])};
      }
      // P = exp2(S * c - lse) of the next half under the dQ and dP MFMAs: RS registers a slot from the second slot after the
      // S MFMAs on, the exponential one slot behind the multiply-add
      if constexpr (n == KK + 1) {
        if (masked_n) mask_half(sc[PAR ^ 1], jn, KTN);
      }
      constexpr int RS = 16 / KK, P0 = KK + 2;
      static_assert(P0 + KK + 1 <= kSlots, "all sixteen registers");
      if constexpr (n >= P0 && n < P0 + KK) {
#pragma unroll
        for (int x = RS * (n - P0); x < RS * (n - P0 + 1); ++x) S2_AT(sc[PAR ^ 1], x) = __builtin_fmaf(S2_AT(sc[PAR ^ 1], x), c, neg_ln[x >> 3]);
      }
      if constexpr (n >= P0 + 1 && n < P0 + KK + 1) {
#pragma unroll
        for (int x = RS * (n - P0 - 1); x < RS * (n - P0); ++x) S2_AT(sc[PAR ^ 1], x) = fast_exp2(S2_AT(sc[PAR ^ 1], x));
      }
      // Nothing to execute: ties the probabilities to this slot.  Their first use is in the next
      // half step, and the optimiser would otherwise collect the arithmetic there, after the last
      // MFMA of this one and out of its shadow.
      if constexpr (n >= P0 && n < P0 + KK + 1)
        asm volatile("" : "+v"(sc[PAR ^ 1][0][0]), "+v"(sc[PAR ^ 1][0][1]), "+v"(sc[PAR ^ 1][1][0]), "+v"(sc[PAR ^ 1][1][1]));
      S2_FENCE();
    });
  };

  // ------------------------------------------------------------------ the loop: one chunk per trip
  // trip ch: half steps (ch, 0) and (ch, 1); chunk ch + 1 is requested at the start of the trip
  // into the other stage (free since the barrier that ended the last trip) and must have landed
  // when the second half step reads its K and V rows
  for (int ch = 0; ch < total; ++ch) {
    const int st = ch & 1;
    if (ch + 1 < total) issue_chunk(row_n, st ^ 1);
    half_step(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, st, st, ch, state_c);
    wait_all_loads();
    __syncthreads();
    half_step(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, st, st ^ 1, min(ch + 1, total - 1), state_n);
    // keeps the entry window moving (entries of chunk ch + 1 on)
    if (!DENSE) (void)list.get(FINE ? min((4 * (ch + 1)) >> ppe_sh, n_ent - 1) : min(ch + 1, total - 1) >> cpb_sh, lane);
    state_c = state_n;
    chunk_at(ch + 2, row_n, state_n);
    __syncthreads();  // every wavefront is done with chunk ch before the next trip loads over it
  }

  // ------------------------------------------------------------------ epilogue
  // dQ = scale * acc goes out through LDS (free since the loop's last barrier; each wavefront uses a
  // region of its own, so no barrier): a lane holds its row's features four at a time, and storing
  // them from there would touch 32 rows per instruction with 16 bytes each; read back 16 bytes per
  // lane, row after row, an instruction stores four whole rows.
  if (!wave_on) return;
  constexpr int RS = D + 8;  // staging row stride (elements)
  uint16_t* stage = sm.k[0] + wave * MW * RS;
  static_assert(4 * MW * RS <= 2 * Tile::kElems, "the staging rows fit the K stages");
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[ft][nt][e] * p.scale);
      *reinterpret_cast<bf16x4*>(stage + (16 * nt + l16) * RS + 16 * ft + 4 * g) = w;
    }
  uint16_t* obase = p.dq + q_off + (int64_t)qw0 * p.q_st;
  constexpr int PPR = D / 8, RPI = 64 / PPR;  // 16-byte pieces per row, rows per instruction
#pragma unroll
  for (int i = 0; i < MW / RPI; ++i) {
    const int r = RPI * i + lane / PPR, piece = lane % PPR;
    const u32x4 x = *reinterpret_cast<const u32x4*>(stage + r * RS + 8 * piece);
    if (!VARLEN || qw0 + r < N) *reinterpret_cast<u32x4*>(obase + (int64_t)r * p.q_st + 8 * piece) = x;
  }
}

#undef S2_AT

}  // namespace s2
