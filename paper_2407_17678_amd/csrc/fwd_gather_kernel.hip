// Forward for mask blocks of 16 and 32 tokens: the same tiles, lists, orientation and hand-written interleave as
// fwd_pipe_kernel.hip, with the keys of a chunk gathered 16 at a time (PieceTile in device_util.h) from the next
// blocks of the tile's list.  A wavefront's 32 query rows are one or two mask rows, and much of what the tile's
// list holds is not theirs (a local window of four blocks of 32 makes a list of seven), so the unit of work is half a
// chunk, 32 keys:
//
//   * The scores of a half run in one stream with the probabilities of the half before it and their contraction
//     with V.  A wavefront leaves the stream out where neither half is its own.  Where one of them is, the scores of the
//     other are replaced by zeros, its probabilities are exactly 0 and its V fragments are read from a few zeros in LDS:
//     what the rows of K and V that are not its own hold does not matter.  (Leaving out just the contraction has
//     the compiler move the accumulators between registers, which costs more.)
//   * Blocks of 16: a half is two blocks.  Where only one of them is mine the same is done for the other.
//   * The scores of a half need its K, the second contraction, a half later, its V: the V tile is staged two
//     pieces behind the K tile, so that both tiles of a trip are used up in it and one barrier a trip is enough.
//   * The running maximum is exact (see fwd_pipe_kernel.hip) and moves by half chunks: relative error of O against 64
//     bits 2.115e-3 (8192 x 64, blocks of 32) and 2.124e-3 (x 128, blocks of 16), by whole chunks 2.126e-3 and 2.133e-3.
//
// Measured (us), against a kernel that walked 32 keys a step phase by phase, and against whole 64-key chunks in the
// loop of fwd_pipe_kernel.hip, in which a wavefront that keeps one half of a chunk computes both: 2 x 9 heads x 6080 x 128,
// blocks of 32, window 3 42 / 48 / 42; 34 x 7136 x 128, blocks of 32, window 3 70 / 81 / 72; 26 x 16064 x 128, window 4 154 / 156 /
// 144; 45 x 12704 x 64, blocks of 16 182 / 144 / 136; 60 x 4864 rows of 34560 x 128, blocks of 16 (nearly every half kept) 667 / 369 /
// 398; packed 11 x 32 x 64, blocks of 32 99 / 124 / 109; 60 x 8192 x 64, blocks of 32, window 4 96 / 111 / 101.  At head_dim 64 it is bound
// by the vector instructions (an exponential takes the time of two), at 128 by those, the matrix pipe and the LDS alike;
// short lists by a tile's start and end, where the first of the three, at head_dim 64, had five workgroups to a compute
// unit (three here: steps of 32 keys would halve the LDS, but four wavefronts to a SIMD spill and measured slower).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "config.h"
#include "device_util.h"
#include "kernels.h"
#include "sched_util.h"

namespace s2 {

namespace {

constexpr float kNegInf = -__builtin_inff();

// VARLEN: a packed batch of sequences of different lengths, as in fwd_pipe_kernel.hip.
template <int D, int S, bool VARLEN>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 3) void fwd_gather_kernel(const AttnParams p) {
  typedef DmaTile<D> Tile;
  typedef PieceTile<D> Piece;
  __shared__ __attribute__((aligned(16))) uint16_t sk[2][Tile::kElems];
  __shared__ __attribute__((aligned(16))) uint16_t sv[2][Tile::kElems];
  __shared__ __attribute__((aligned(16))) uint16_t zeros[32 * (D / 32)];  // as far as the offsets of a V fragment group reach
  constexpr int BM = kFwdBM, MW = 32;
  constexpr int KK = D / 16, DT = D / 32;
  constexpr int NS = 2 * KK;  // MFMAs of a half: KK of the scores, 2 * DT of the second contraction
  constexpr int NG = Piece::kGroups;
  constexpr int RB = Tile::kStride * 2;  // bytes per tile row
  constexpr int kLead = D == 128 ? 5 : 3, kRing = kLead + 1;
  constexpr int PPB = S / 16, EPC = 4 / PPB;  // pieces of a block, list entries of a chunk
  static_assert(2 * DT == KK && (S == 16 || S == 32), "");

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
  if (whole) {
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
  const int qw0 = tile * BM + wave * MW;    // first query row of this wavefront (sequence position)
  const int ql0 = qw0 - p.q_row0;           // the same as a row of q / o / lse
  const bool wave_on = ql0 < n_q;           // whether I have query rows at all

  const int64_t q_off = (VARLEN ? row_base * p.q_st : b * p.q_sb) + h * p.q_sh;
  const int64_t kv_off = (VARLEN ? row_base * p.kv_st : b * p.kv_sb) + h * p.kv_sh;
  // minus the bias the grouped direct loads put into their lane offsets
  const uint16_t* kb = p.k + kv_off - Piece::kBias / 2;
  const uint16_t* vb = p.v + kv_off - Piece::kBias / 2;

  if (!whole) {
    ent_lo = load_const<int32_t>(p.q_tiles.ptr + h * T + tile);
    n_ent = load_const<int32_t>(p.q_tiles.ptr + h * T + tile + 1) - ent_lo;
  }
  const int total = (n_ent + EPC - 1) / EPC;  // chunks
  if (total <= 0) return;
  EntryList list;
  list.init(p.q_tiles.ent + ent_lo, n_ent, lane);

  // Q^T fragments stay in registers for the whole tile (B operands of the score MFMAs); a lane without
  // a row of its own reads the last row, its result is never stored
  bf16x8 qf[KK];
  const int q_lane = min(ql0 + l32, n_q - 1);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    qf[kk] = *reinterpret_cast<const bf16x8*>(p.q + q_off + (int64_t)q_lane * p.q_st + 16 * kk + 8 * half);

  // Entry i of the list (0 after its end: the first block, kept by nobody); its first key row; which of my
  // two groups of 16 query rows keep it (bits 0 and 1; both or neither for blocks of 32).
  auto row_of = [&](uint32_t e) S2_INLINE { return (int)(e >> 16) * S; };
  auto bits_of = [&](uint32_t e) S2_INLINE { return S == 32 ? (int)((e >> wave) & 1) * 3 : (int)(e >> (2 * wave)) & 3; };
  // What this wavefront needs to know of a chunk: the first key rows of the pieces it fetches for the K tile and
  // for the V tile (which lags by two pieces: the chunk's second half comes with the next chunk's first), and of
  // either half which pieces are mine (two bits), and whether some of it is masked for some of my rows.
  struct Chunk {
    int k_row, v_row, on0, on1, masked0, masked1;
  };
  const uint32_t late_from = (uint32_t)(qw0 / S) << 16;  // entries from my first row's block on
  auto chunk_at = [&](int j) S2_INLINE {
    Chunk c;
    const int i0 = EPC * j;
    const int src = (i0 >> 6) != list.batch ? list.nxt : list.cur;  // a chunk's entries are of one batch
    c.k_row = row_of(__builtin_amdgcn_readlane(src, (i0 + wave / PPB) & 63)) + (PPB == 2 ? 16 * (wave & 1) : 0);
    c.v_row = row_of(__builtin_amdgcn_readlane(src, (i0 + (wave ^ 2) / PPB) & 63)) + (PPB == 2 ? 16 * (wave & 1) : 0);
    // every lane's entry at once, then the chunk's bits
    const int bits = bits_of(src);
    const uint32_t any = (uint32_t)(__ballot(bits != 0) >> (i0 & 63));
    const uint32_t whole = (uint32_t)((__ballot(bits == 3) & ~__ballot((uint32_t)src >= late_from)) >> (i0 & 63));
    if constexpr (S == 32) {
      c.on0 = any & 1 ? 3 : 0;
      c.on1 = any & 2 ? 3 : 0;
      c.masked0 = !(whole & 1);
      c.masked1 = !(whole & 2);
    } else {
      c.on0 = any & 3;
      c.on1 = (any >> 2) & 3;
      c.masked0 = (whole & 3) != 3;
      c.masked1 = ((whole >> 2) & 3) != 3;
    }
    if (!wave_on) c.on0 = c.on1 = 0;
    if (VARLEN) {
      c.k_row = min(c.k_row, N - 1);
      c.v_row = min(c.v_row, N - 1);
    }
    return c;
  };

  f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = f32x16{};
  float m_ref = kNegInf;  // running maximum (raw scores) of my query
  float mc = 0.f;         // the same times scale * log2(e); 0 while nothing was seen
  float l_run = 0.f;      // sum of the probabilities over my half's key rows
  const float c = p.scale_log2e;
  // Lane offsets of my direct loads, for K and for V.  Where a packed sequence ends inside the rows I fetch
  // (VARLEN) they are limited to the rows that exist; the lists ascend, so from then on every piece is such
  // a piece, with fewer and fewer rows.
  typename Piece::Plan plan_k = Piece::plan(p.kv_st, lane), plan_v = plan_k;
  auto issue_k = [&](int row, int stage) S2_INLINE {
    if (VARLEN && row + 16 > N) Piece::limit(plan_k, N - row, p.kv_st);
    static_for<NG>([&](auto gc) S2_INLINE { Piece::template issue<decltype(gc)::value>(plan_k, kb + (int64_t)row * p.kv_st, sk[stage], wave); });
  };
  auto issue_v = [&](int row, int stage) S2_INLINE {
    if (VARLEN && row + 16 > N) Piece::limit(plan_v, N - row, p.kv_st);
    static_for<NG>([&](auto gc) S2_INLINE {
      Piece::template issue<decltype(gc)::value>(VARLEN ? plan_v : plan_k, vb + (int64_t)row * p.kv_st, sv[stage], wave);
    });
  };
  const uint32_t k_lane = lds_addr(sk[0]) + l32 * RB + 16 * half, v_lane = lds_addr(sv[0]) + 2 * Tile::tr_base(lane);

  // drops what my query does not see of half kt of chunk j: keys after it and pieces its mask row does not keep
  auto mask_half = [&](f32x16& s, int j, int kt) S2_INLINE {
    const int qpos = qw0 + l32;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t e = (uint32_t)list.peek(EPC * j + (2 * kt + u) / PPB);
      // how many of the piece's keys I see, counted from the first one my half of the wavefront holds
      int lim = qpos - (row_of(e) + (PPB == 2 ? 16 * u : 0)) + 1 - 4 * half;
      if (S == 16 && !((bits_of(e) >> (l32 >> 4)) & 1)) lim = -4;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (8 * (i >> 2) + (i & 3) >= lim) s[8 * u + i] = kNegInf;
    }
  };
  auto max_part = [&](int r0, int r1, const f32x16& s, float& mx) S2_INLINE {
#pragma unroll
    for (int r = r0; r < r1; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);
  };
  // The maximum of a half's scores (mx, unless some are masked) against the running one, and what has been
  // accumulated so far to the new one.  (A lane that has seen no key yet has m_ref = -inf, and while it sees none
  // mx is no larger.)
  auto finish_scores = [&](f32x16& s, int j, int kt, bool masked, float mx) S2_INLINE {
    if (masked) {
      mask_half(s, j, kt);
      mx = kNegInf;
      max_part(0, 16, s, mx);
      mx = max_halves(mx);
    }
    if (__any(mx > m_ref)) {
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

  // Scores of two halves, one of each parity: register r is key 8 * (r / 4) + 4 * half + r % 4 of the half, lane % 32
  // the query; then its probabilities, in place.
  f32x16 s0 = f32x16{}, s1 = f32x16{};

  // One half step of trip t: the scores of half H of chunk t (into sn), and the second contraction of the half
  // before it (whose scores are in sc and whose V rows are half H of the V tile).  on_c, on_n: which pieces of that
  // one and of this one are mine.
  auto half_step = [&](auto hc, int t, int on_c, int on_n, int masked, f32x16& sc, f32x16& sn) S2_INLINE {
    constexpr int H = decltype(hc)::value;
    float mx = kNegInf;
    if ((on_c | on_n) != 0) {
      const uint32_t stage = (t & 1) * (uint32_t)Tile::kBytes;
      uint32_t k_row = k_lane + stage;
      // where the V fragments of either slab are read from, their first and their last eight rows
      uint32_t v_tr[2][2];
#pragma unroll
      for (int i = 0; i < 4; ++i) v_tr[i >> 1][i & 1] = v_lane + (stage + (32 * H + 8 * i) * RB);
      float mc_use = mc;
      if (on_c != 3) {
        const uint32_t z0 = lds_addr(zeros);
        if (!(on_c & 1)) v_tr[0][0] = v_tr[0][1] = z0;
        if (!(on_c & 2)) v_tr[1][0] = v_tr[1][1] = z0;
        if (on_c == 0) mc_use = __builtin_inff();  // (not mine: its scores are zeros, its probabilities 0)
      }
      asm volatile("" : "+v"(k_row), "+v"(v_tr[0][0]), "+v"(v_tr[0][1]), "+v"(v_tr[1][0]), "+v"(v_tr[1][1]), "+v"(mc_use));
      bf16x8 fr[kRing];
      u32x4 pb[2];
      // fragment f: KK row fragments of K, then the transposed fragments of V (16-key slab, feature tile)
      auto frag_load = [&](auto fc) S2_INLINE {
        constexpr int f = decltype(fc)::value;
        if constexpr (f < KK)
          fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read16(k_row, 32 * H * RB + 32 * f));
        else
          fr[f % kRing] = __builtin_bit_cast(bf16x8, lds_read_tr2(v_tr[(f - KK) / DT][0], v_tr[(f - KK) / DT][1], 64 * ((f - KK) % DT), 64 * ((f - KK) % DT)));
      };
      // Probabilities in three stages - scale and shift, exponential, sum and pack - each a slot behind the one
      // before it: eight elements every five slots (D = 64: four a slot), so that slab u is packed before slot
      // KK + DT * u, where its MFMAs start.
      constexpr auto upto = [](int sl) { return std::max(0, std::min(16, D == 128 ? 8 * (sl + 1) / 5 : 4 * (sl + 1))); };
      static_assert(upto(KK - 3) >= 8 && upto(KK + DT - 3) >= 16, "packed in time");
      static_for<kLead>([&](auto fc) S2_INLINE { frag_load(fc); });
      S2_FENCE();
      static_for<NS>([&](auto nc) S2_INLINE {
        constexpr int n = decltype(nc)::value;
        if constexpr (n + kLead < NS) frag_load(std::integral_constant<int, n + kLead>{});
        if constexpr (n < KK)
          sn = mfma32(fr[n % kRing], qf[n], n == 0 ? f32x16{} : sn);
        else
          acc[(n - KK) % DT] = mfma32(fr[n % kRing], __builtin_bit_cast(bf16x8, pb[(n - KK) / DT]), acc[(n - KK) % DT]);
#pragma unroll
        for (int r = upto(n - 1); r < upto(n); ++r) sc[r] = __builtin_fmaf(sc[r], c, -mc_use);
#pragma unroll
        for (int r = upto(n - 2); r < upto(n - 1); ++r) sc[r] = fast_exp2(sc[r]);
#pragma unroll
        for (int r = upto(n - 3); r < upto(n - 2); ++r) {
          l_run += sc[r];  // (the unrounded probabilities, see fwd_pipe_kernel.hip)
          if (r & 1) pb[r >> 3][(r & 7) >> 1] = pack2(sc[r - 1], sc[r]);
        }
        // maximum of the new scores, once their MFMAs are done
        constexpr int M0 = D == 128 ? KK + 2 : KK + 1, kMax = D == 128 ? 4 : 8;
        static_assert((NS - 1 - M0) * kMax >= 16, "all sixteen registers and a slot for the other half's");
        if constexpr (n >= M0 && kMax * (n - M0) < 16) max_part(kMax * (n - M0), std::min(16, kMax * (n - M0 + 1)), sn, mx);
        if constexpr (n == NS - 1) mx = max_halves(mx);
        // Nothing to execute: ties the running sum and maximum to this slot, or the optimiser collects their
        // additions and comparisons after the last MFMA.
        asm volatile("" : "+v"(l_run), "+v"(mx));
        S2_FENCE();
      });
    }
    if (on_n)
      finish_scores(sn, t, H, masked, mx);
    else
      sn = f32x16{};
  };

  // Trip t: the scores of chunk t, the second contraction of the halves 2 t - 1 and 2 t; meanwhile the K
  // tile of chunk t + 1 and the V tile of its trip are fetched.
  if (tid < 8 * DT) reinterpret_cast<uint64_t*>(zeros)[tid] = 0;
  Chunk cur = chunk_at(0);
  issue_k(cur.k_row, 0);
  if (wave >= 2) issue_v(cur.v_row, 0);  // (there are no keys before the first)
  int on_c = 0, v_lag = cur.v_row;
  wait_all_loads();
  __syncthreads();
  for (int t = 0; t <= total; ++t) {
    const Chunk nxt = chunk_at(t + 1);
    if (t < total) {
      if (t + 1 < total) issue_k(nxt.k_row, (t + 1) & 1);
      issue_v(wave < 2 ? v_lag : nxt.v_row, (t + 1) & 1);
    }
    half_step(std::integral_constant<int, 0>{}, t, on_c, cur.on0, cur.masked0, s1, s0);
    half_step(std::integral_constant<int, 1>{}, t, cur.on0, cur.on1, cur.masked1, s0, s1);
    on_c = cur.on1;
    v_lag = nxt.v_row;
    (void)list.get(EPC * (t + 1), lane);  // keeps the entry window moving (entries of chunk t + 1 on)
    cur = nxt;
    wait_all_loads();
    __syncthreads();
  }

  if (!wave_on) return;
  const float l_tot = sum_halves(l_run);
  store_rows<D, VARLEN>(acc, 1.0f / l_tot, sk[0] + wave * MW * (D + 8), p.o + q_off + (int64_t)ql0 * p.q_st, p.q_st, n_q - ql0, lane);
  const int64_t lse_row = VARLEN ? (int64_t)h * p.seqlen + row_base + ql0 + l32  // [heads, rows of the tensors]
                                 : ((int64_t)b * p.heads + h) * p.q_rows + ql0 + l32;
  if (half == 0 && (!VARLEN || ql0 + l32 < n_q)) p.lse[lse_row] = m_ref * p.scale + __logf(l_tot);
}

template <int D, int S>
hipError_t launch_one(const AttnParams& p, hipStream_t stream) {
  const dim3 grid(p.row_map.grid()), block(kThreads);
  if (p.cu_seqlens)
    hipLaunchKernelGGL((fwd_gather_kernel<D, S, true>), grid, block, 0, stream, p);
  else
    hipLaunchKernelGGL((fwd_gather_kernel<D, S, false>), grid, block, 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_gather(const AttnParams& p, hipStream_t stream) {
  if (p.head_dim == 128) return p.block_size == 16 ? launch_one<128, 16>(p, stream) : launch_one<128, 32>(p, stream);
  return p.block_size == 16 ? launch_one<64, 16>(p, stream) : launch_one<64, 32>(p, stream);
}

}  // namespace s2
