// dQ kernel: the row-stationary half of the backward pass (the gradient of the forward of section 3.2).
// Same tiles, lists, staging and orientation as the forward (fwd_pipe_kernel.hip) - a workgroup owns 128
// query rows, a wavefront 32 of them, and walks the 64-key chunks of the KV blocks its mask rows keep,
// recomputing P and forming dS = P * (dP - delta), dQ += scale * dS K; it also computes
// delta = rowsum(dO * O) and leaves the row statistics in the workspace for the dK/dV
// kernel - with a hand-scheduled inner loop:
//
//   * it runs in half chunks of 32 keys, skewed by one half: S and dP of the next half are computed
//     around the dQ MFMAs of this one, with this half's dS arithmetic under the former and the next
//     half's exponentials under the latter;
//   * the order is written out, one MFMA per slot with its share of the vector work, LDS reads and
//     direct loads, and fenced so that the compiler keeps it (see sched_util.h for the measurements
//     behind this); the A operands pass through a ring of registers requested a few MFMAs ahead;
//   * the direct loads of a tile are issued two or three to a write of M0.
//
// Head_dim 64, mask blocks below 64 tokens (FINE: chunks gathered from 16-key pieces) and ragged ends
// (VARLEN) are the same loop, as in the forward.  Against the phase-by-phase kernel that these used to run,
// per launch: 2 x 16 heads x 4096 x 64, blocks of 64: 50.1 -> 45.9 us; 2 x 16 x 3904 x 128 (61 blocks):
// 73.3 -> 65.2 us; 1 x 16 x 8192 x 128, blocks of 16: 84.2 -> 70 us; a packed batch of 8 sequences of 200 to
// 8192 rows x 32 heads: 497 us in two launches -> 478 us in one.  It is bound as the forward is: by the
// matrix pipe and the vector work beside it over long lists, by a tile's start and end over short ones.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "config.h"
#include "device_util.h"
#include "kernels.h"
#include "sched_util.h"

namespace s2 {

namespace {

constexpr float kNegInf = -__builtin_inff();
constexpr float kLog2e = 1.4426950408889634f;

template <int D>
struct DqPipeSmem {
  uint16_t k[2][DmaTile<D>::kElems];
  uint16_t v[2][DmaTile<D>::kElems];
};

template <int D, bool DENSE, bool FINE, bool VARLEN>
__global__ __launch_bounds__(kThreads, 2) void dq_pipe_kernel(const AttnParams p) {
  typedef DmaTile<D> Tile;
  typedef PieceTile<D> Piece;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  DqPipeSmem<D>& sm = *reinterpret_cast<DqPipeSmem<D>*>(smem_raw);
  constexpr int BM = kBwdBM, MW = 32, CH = 64;
  constexpr int KK = D / 16, DT = D / 32;
  constexpr int NG = Piece::kGroups;
  constexpr int RB = Tile::kStride * 2;  // bytes per tile row
  constexpr int kSlots = 3 * KK;         // MFMAs (and fragments) per half step: KK of S, 2 * DT of dQ, KK of dP
  constexpr int kLead = D == 128 ? 5 : 3, kRing = kLead + 1;  // (at D = 128 3 to 7 measure the same)
  static_assert(2 * DT == KK, "the dQ part is as long as the S and dP parts");
  static_assert(!(DENSE && (FINE || VARLEN)), "the dense form walks 64-key blocks of whole sequences");

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  if (!DENSE && !VARLEN) clear_split_counts(p, blockIdx.x * kThreads + tid);
  const int T = p.q_tiles.tiles_per_head;
  const int T_run = VARLEN ? (p.q_rows + BM - 1) / BM : T;  // packed batch: tiles of the longest length allowed
  int bh, rank;
  if (!map_workgroup(blockIdx.x, p.batch * p.heads, T_run, p.map_group, bh, rank)) return;
  const int b = bh / p.heads, h = bh - b * p.heads;
  int tile = DENSE ? (T - 1 - rank) : VARLEN ? 0 : p.q_tiles.order[h * T + rank];
  int N = p.seqlen, row_base = 0;  // my sequence's length, and the rows of the tensors before it
  if (VARLEN) {
    const int lo = p.cu_seqlens[b], hi = p.cu_seqlens[b + 1];
    row_base = min(max(lo, 0), p.seqlen);  // whatever the array holds, stay inside the tensors
    N = min(min(max(hi - lo, 0), p.q_rows), p.seqlen - row_base);
    const int T_seq = (N + BM - 1) / BM;
    if (rank >= T_seq) return;
    tile = T_seq - 1 - rank;
  }
  const int S = DENSE ? CH : p.block_size;  // FINE: 16 or 32, else 64 or 128
  const int cpb_sh = S == 128 ? 1 : 0, cpb_m = (1 << cpb_sh) - 1;  // chunks per list entry
  const int ppe_sh = S == 32 ? 1 : 0;                              // FINE: 16-key pieces per list entry
  const int qw0 = tile * BM + wave * MW;  // first query row of this wavefront
  const bool wave_on = qw0 < N;           // whether I have query rows at all
  const int my_member = (qw0 / S) - tile * (BM / S);

  const int64_t q_off = (VARLEN ? row_base * p.q_st : b * p.q_sb) + h * p.q_sh;
  const int64_t kv_off = (VARLEN ? row_base * p.kv_st : b * p.kv_sb) + h * p.kv_sh;
  // minus the bias the grouped direct loads put into their lane offsets
  const uint16_t* kb = p.k + kv_off - Piece::kBias / 2;
  const uint16_t* vb = p.v + kv_off - Piece::kBias / 2;

  int ent_lo = 0, n_ent;
  if (DENSE) {
    n_ent = min(N, (tile + 1) * BM) / CH;
  } else {
    ent_lo = p.q_tiles.ptr[h * T + tile];
    n_ent = p.q_tiles.ptr[h * T + tile + 1] - ent_lo;
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
      j = min(j, total - 1);
      int kv0;
      bool keep = true;
      if (DENSE) {
        kv0 = j * CH;
      } else {
        const int e = list.peek(j >> cpb_sh);
        kv0 = (e >> 16) * S + (j & cpb_m) * CH;
        keep = (e >> my_member) & 1;
      }
      row = kv0 + 16 * wave;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        if (keep && kv0 + 32 * kt <= qw0 + MW - 1) state |= 1 << kt;
        if (kv0 + 32 * kt + 31 > qw0) state |= 4 << kt;
      }
    }
    if (!inside || !wave_on) state &= ~3;
    if (VARLEN) row = min(row, N - 1);
  };

  typename Piece::Plan plan = Piece::plan(p.kv_st, lane);
  auto issue_chunk = [&](int row, int stage) S2_INLINE {
    // where a packed sequence ends inside the rows I fetch they are limited to the rows that exist; the
    // lists ascend, so from then on every piece is such a piece, with fewer and fewer rows
    if (VARLEN && row + 16 > N) Piece::limit(plan, N - row, p.kv_st);
    const uint16_t* kg = kb + (int64_t)row * p.kv_st;
    const uint16_t* vg = vb + (int64_t)row * p.kv_st;
    static_for<NG>([&](auto gc) S2_INLINE {
      constexpr int g = decltype(gc)::value;
      Piece::template issue<g>(plan, kg, sm.k[stage], wave);
      Piece::template issue<g>(plan, vg, sm.v[stage], wave);
    });
  };
  int row_n, state_c, state_n;
  {
    int row_c;
    chunk_at(0, row_c, state_c);
    chunk_at(1, row_n, state_n);
    issue_chunk(row_c, 0);
  }

  // Q^T and dO^T fragments (B operands), lane = query; delta = rowsum(dO * O) of my query from the
  // dO fragments (my half of the row's features, then the two halves added), written out with LSE
  // as the dK/dV kernel, which runs after this one, wants them.  A lane without a row of its own
  // reads the last row; nothing of it is stored.
  bf16x8 qf[KK], gf[KK];
  float part = 0.f;
  const int my_row = min(qw0 + l32, N - 1);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int64_t o = q_off + (int64_t)my_row * p.q_st + 16 * kk + 8 * half;
    qf[kk] = *reinterpret_cast<const bf16x8*>(p.q + o);
    gf[kk] = *reinterpret_cast<const bf16x8*>(p.d_o + o);
    const bf16x8 of = *reinterpret_cast<const bf16x8*>(p.o + o);
#pragma unroll
    for (int e = 0; e < 8; ++e) part = __builtin_fmaf((float)gf[kk][e], (float)of[e], part);
  }
  const float delta_l = sum_halves(part);
  const int64_t stat_row = VARLEN ? (int64_t)h * p.seqlen + row_base + my_row  // [heads, rows of the tensors]
                                  : ((int64_t)b * p.heads + h) * N + my_row;
  const float lse_l = p.lse[stat_row] * kLog2e;
  if (half == 0 && qw0 + l32 < N) {
    p.neg_delta[stat_row] = -delta_l;
    p.neg_lse[stat_row] = p.lse[stat_row] * p.neg_inv_scale;
  }

  f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = f32x16{};
  const float c = p.scale_log2e;
  // lane parts of the addresses the fragments are read at (stage 0 of K; V lies v_from_k further on)
  const uint32_t k_lane = lds_addr(sm.k[0]) + l32 * RB + 16 * half, tr_lane = lds_addr(sm.k[0]) + 2 * Tile::tr_base(lane);
  constexpr uint32_t v_from_k = sizeof(sm.k);

  // Scores of a 32-key half: register r is key 8 * (r / 4) + 4 * half + r % 4 of the half, lane % 32
  // the query.  sc holds S, then P in place; dp holds dP, then dS in place.
  f32x16 sc[2], dp;  // sc[parity of the half]
  u32x4 dsb[2];      // dS of this half as B operands [16-key slab]

  // Drops what my query does not see of half kt of chunk j: keys after it and (FINE) pieces its mask row
  // does not keep.  (A half that is not mine at all gets lse = +inf instead: P = dS = 0.)
  auto mask_half = [&](f32x16& s2, int j, int kt) S2_INLINE {
    const int qpos = qw0 + l32;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      int row, bits = 3;
      if constexpr (FINE) {
        piece_at(j, 2 * kt + u, row, bits);
      } else if (DENSE) {
        row = j * CH + 32 * kt + 16 * u;
      } else {
        row = (list.peek(j >> cpb_sh) >> 16) * S + (j & cpb_m) * CH + 32 * kt + 16 * u;
      }
      // how many of the piece's keys I see, counted from the first one my half of the wavefront holds
      int lim = qpos - row + 1 - 4 * half;
      if (FINE && !((bits >> (l32 >> 4)) & 1)) lim = -4;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (8 * (i >> 2) + (i & 3) >= lim) s2[8 * u + i] = kNegInf;
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
    sc[0] = f32x16{};
    dp = f32x16{};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      sc[0] = mfma32(__builtin_bit_cast(bf16x8, lds_read16(k_row, 32 * kk)), qf[kk], sc[0]);
      dp = mfma32(__builtin_bit_cast(bf16x8, lds_read16(v_row, 32 * kk)), gf[kk], dp);
    }
    act_cur = state_c & 1;
    on_cur = (state_c >> 4) & 3;
    if (state_c & 4) mask_half(sc[0], 0, 0);
    const float l0 = act_cur ? lse_l : __builtin_inff();
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[0][r] = fast_exp2(__builtin_fmaf(sc[0][r], c, -l0));
    if (!act_cur || (FINE && on_cur != 3)) {  // (what does not come from a piece of mine may not be a number)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (!act_cur || !((on_cur >> (r >> 3)) & 1)) sc[0][r] = dp[r] = 0.f;
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
      sc[PAR ^ 1] = f32x16{};
      dp = f32x16{};
      return;
    }
    const uint32_t from_n = stn * (uint32_t)Tile::kBytes + 32 * KTN * RB, from_this = stc * (uint32_t)Tile::kBytes + 32 * KT * RB;
    const uint32_t row_off = act_n ? from_n : from_this, tr_off = act_this ? from_this : from_n;
    uint32_t k_row = k_lane + row_off, k_tr = tr_lane + tr_off, k_tr1 = k_tr;
    if constexpr (FINE) {
      const int on_r = act_n ? on_n : on_this, on_t = act_this ? on_this : on_n;
      if (on_r != 3) k_row += (on_r == 1 ? 0 : 16 * RB) - (l32 >> 4) * 16 * RB;
      if (on_t != 3) {
        if (on_t == 2) k_tr += 16 * RB;
        k_tr1 = k_tr - 16 * RB;
      }
    }
    uint32_t v_row = k_row + v_from_k;
    asm volatile("" : "+v"(k_row), "+v"(v_row), "+v"(k_tr));
    if constexpr (FINE) asm volatile("" : "+v"(k_tr1));
    bf16x8 fr[kRing];
    // fragment f of the half step, in the order the MFMAs use them: KK row fragments of the next
    // half's K, KK transposed fragments of this half's K (16-key slab, feature tile), KK row fragments
    // of the next half's V
    auto frag_load = [&](auto fc) S2_INLINE {
      constexpr int f = decltype(fc)::value;
      if constexpr (f < KK)
        fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read16(k_row, 32 * f));
      else if constexpr (f < 2 * KK)
        fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read_tr(FINE && f - KK >= DT ? k_tr1 : k_tr, 16 * ((f - KK) / DT) * RB + 64 * ((f - KK) % DT), RB));
      else
        fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read16(v_row, 32 * (f - 2 * KK)));
    };
    static_for<kLead>([&](auto fc) S2_INLINE { frag_load(fc); });
    const float ln = act_n ? lse_l : __builtin_inff();
    S2_FENCE();
    static_for<kSlots>([&](auto nc) S2_INLINE {
      constexpr int n = decltype(nc)::value;
      if constexpr (n + kLead < kSlots) frag_load(std::integral_constant<int, n + kLead>{});
      // the MFMA of the slot
      if constexpr (n < KK)  // S of the next half
        sc[PAR ^ 1] = mfma32(fr[n % kRing], qf[n], n == 0 ? f32x16{} : sc[PAR ^ 1]);
      else if constexpr (n < 2 * KK)  // dQ of this half: slab, feature tile
        acc[(n - KK) % DT] = mfma32(fr[n % kRing], __builtin_bit_cast(bf16x8, dsb[(n - KK) / DT]), acc[(n - KK) % DT]);
      else  // dP of the next half
        dp = mfma32(fr[n % kRing], gf[n - 2 * KK], n == 2 * KK ? f32x16{} : dp);
      // dS = P * (dP - delta) of this half under the S MFMAs: RS registers a slot, a slab packed in the
      // slot after its last one
      constexpr int RS = 16 / KK;
      if constexpr (n < KK) {
#pragma unroll
        for (int r = RS * n; r < RS * (n + 1); ++r) dp[r] = sc[PAR][r] * (dp[r] - delta_l);
      }
      if constexpr (n == KK / 2 || n == KK) {
        constexpr int u = n == KK / 2 ? 0 : 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) dsb[u][i] = pack2(dp[8 * u + 2 * i], dp[8 * u + 2 * i + 1]);
      }
      // P = exp2(S * c - lse) of the next half under the dQ and dP MFMAs: RS registers a slot from the second slot after the
      // S MFMAs on, the exponential one slot behind the multiply-add
      if constexpr (n == KK + 1) {
        if (masked_n) mask_half(sc[PAR ^ 1], jn, KTN);
      }
      constexpr int P0 = KK + 2;
      static_assert(P0 + KK + 1 <= kSlots, "all sixteen registers");
      if constexpr (n >= P0 && n < P0 + KK) {
#pragma unroll
        for (int r = RS * (n - P0); r < RS * (n - P0 + 1); ++r) sc[PAR ^ 1][r] = __builtin_fmaf(sc[PAR ^ 1][r], c, -ln);
      }
      if constexpr (n >= P0 + 1 && n < P0 + KK + 1) {
#pragma unroll
        for (int r = RS * (n - P0 - 1); r < RS * (n - P0); ++r) sc[PAR ^ 1][r] = fast_exp2(sc[PAR ^ 1][r]);
      }
      // Nothing to execute: ties the probabilities to this slot.  Their first use is in the next
      // half step, and the optimiser would otherwise collect the arithmetic there, after the last
      // MFMA of this one and out of its shadow.
      if constexpr (n >= P0 && n < P0 + KK + 1) asm volatile("" : "+v"(sc[PAR ^ 1]));
      S2_FENCE();
    });
  };

  // ------------------------------------------------------------------ the loop: one chunk per trip
  // trip ch: half steps (ch, 0) and (ch, 1); chunk ch + 1 is requested at the start of the trip
  // into the other stage (free since the barrier that ended the last trip) and must have landed
  // when the second half step reads its K and V rows
  for (int ch = 0; ch < total; ++ch) {
    const int st = ch & 1;
    issue_chunk(row_n, st ^ 1);  // past the end of the list: the last chunk once more
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
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[dt][4 * g + e] * p.scale);
      *reinterpret_cast<bf16x4*>(stage + l32 * RS + 32 * dt + 8 * g + 4 * half) = w;
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

// A kernel's dynamic LDS limit is a per-device attribute: remember, per device, that it is set.
constexpr int kMaxDevices = 64;
std::atomic<unsigned char> g_smem_set[10][kMaxDevices];

template <int D, bool DENSE, bool FINE, bool VARLEN>
hipError_t launch_one(const AttnParams& p, hipStream_t stream) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < kMaxDevices;
  constexpr int which = (D == 128 ? 5 : 0) + (DENSE ? 4 : FINE + 2 * VARLEN);
  if (!tracked || !g_smem_set[which][dev].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&dq_pipe_kernel<D, DENSE, FINE, VARLEN>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(DqPipeSmem<D>));
    if (e != hipSuccess) return e;
    if (tracked) g_smem_set[which][dev].store(1, std::memory_order_release);
  }
  const int grid = grid_for(p.batch * p.heads, VARLEN ? (p.q_rows + kBwdBM - 1) / kBwdBM : p.q_tiles.tiles_per_head);
  hipLaunchKernelGGL((dq_pipe_kernel<D, DENSE, FINE, VARLEN>), dim3(grid), dim3(kThreads), sizeof(DqPipeSmem<D>), stream, p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_dim(const AttnParams& p, bool dense, hipStream_t stream) {
  if (dense) return launch_one<D, true, false, false>(p, stream);
  if (p.block_size < 64) return p.cu_seqlens ? launch_one<D, false, true, true>(p, stream) : launch_one<D, false, true, false>(p, stream);
  return p.cu_seqlens ? launch_one<D, false, false, true>(p, stream) : launch_one<D, false, false, false>(p, stream);
}

}  // namespace

hipError_t launch_dq(const AttnParams& p, bool dense, hipStream_t stream) {
  return p.head_dim == 128 ? launch_dim<128>(p, dense, stream) : launch_dim<64>(p, dense, stream);
}

}  // namespace s2
