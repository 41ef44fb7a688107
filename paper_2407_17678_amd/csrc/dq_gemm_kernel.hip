// dQ launch of the backward that keeps dS (head_dim 128, mask blocks of 64 or 128 tokens): the
// dK/dV kernel, which runs first, has left dS = P * (dP - delta) in the workspace, rounded to bf16
// exactly as its own dK contraction takes it, so what remains of the gradient of section 3.2's
// forward on the query side is the single contraction dQ = scale * dS K over the kept blocks -
// nothing is recomputed (the row-stationary kernel in dq_pipe_kernel.hip forms S and dP a second time
// to get at dS).
//
// A workgroup owns 128 query rows and walks the 64-key chunks of the KV blocks its mask rows keep,
// as the other row-stationary kernels do.  Its four wavefronts split a chunk two by two: 64 query
// rows (one dS unit) x 32 keys each, so that every transposed K fragment read from LDS feeds two
// MFMAs - the kernel would otherwise be bound by the rate at which LDS takes instructions - and the
// two key halves are added through LDS when the tile is done.  Per chunk the K rows are staged for
// all four wavefronts and, per wavefront, the 4 KiB of dS that are its own: the dK/dV kernel wrote
// dS with the key on the lane, here the query has to be, so the pieces go through LDS and come back
// through the transpose read.  What bounds the kernel then is the one pass over dS in HBM (2 bytes
// per unmasked pair and 128 flop against it).
//
// dS in the workspace: units of 64 queries x 64 keys, 8 KiB each, found through AttnParams::dq_units;
// inside a unit [32-key half][32-query half][key][g = 0..3][8 queries as the writing lane held them: 4 * g + 0..3, then
// 16 + 4 * g + 0..3].
#include <hip/hip_runtime.h>

#include "config.h"
#include "device_util.h"
#include "kernels.h"
#include "sched_util.h"
#include "smem_limit.h"

namespace s2 {

namespace {

// One wavefront's dS of a chunk in LDS as it lies in the unit, 64 bytes a key, but 4 keys (256 bytes) at every kDsQuadStride: the
// four 16-lane groups of a transpose read, 4 keys each, then fall on different banks (each touches 8 of every 16 bytes).
constexpr int kDsQuadStride = 256 + 32;
constexpr int kDsWaveBytes = 16 * kDsQuadStride;

template <int D>
struct DqGemmSmem {
  union {
    struct {
      uint16_t k[2][ChunkTile<D>::kElems];  // K rows of a chunk, two stages
      unsigned char ds[4][kDsWaveBytes];         // per wavefront: its dS of the current chunk
    } loop;
    float reduce[2][64 * D];  // after the loop: the second key half's sums, per 64-row half of the tile
  };
};

// The loads go through registers (plain loads the compiler tracks, two chunks in flight per
// wavefront, each 4 x 16 bytes of K and 4 x 16 bytes of dS per lane) rather than straight into LDS:
// the kernel lives on bytes in flight, registers are what it has plenty of, and with every load
// tracked the compiler's counted waits let the later chunks stay outstanding.
template <int D>
__global__ __launch_bounds__(kThreads, 2) void dq_gemm_kernel(const AttnParams p) {
  typedef ChunkTile<D> Tile;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  DqGemmSmem<D>& sm = *reinterpret_cast<DqGemmSmem<D>*>(smem_raw);
  constexpr int BM = kBwdBM, FT = D / 16;
  static_assert(D == 128, "a chunk's K rows are 4 x 16 bytes per lane of the workgroup");

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l16 = lane & 15, g = lane >> 4;
  int bh, rank;
  if (!map_workgroup(p.row_map, blockIdx.x, bh, rank)) return;
  const int b = bh / p.by_heads, h = bh - b * p.heads;
  const DevTiles::RowRec rec = p.q_tiles.row_rec(h, rank);
  const int tile = rec.tile;
  const int S = p.block_size;  // 64 or 128
  const int cpb_sh = S == 128 ? 1 : 0, cpb_m = (1 << cpb_sh) - 1;
  const int qhalf = wave >> 1;             // which 64-row half of the tile: one dS unit per chunk
  const int khalf = wave & 1;              // which 32 keys of the chunk
  const int q0 = tile * BM + 64 * qhalf;   // first query row of this wavefront

  const int64_t q_off = b * p.q_sb + h * p.q_sh;
  const uint16_t* kb = p.k + b * p.kv_sb + h * p.kv_sh;
  const unsigned char* ds_b = reinterpret_cast<const unsigned char*>(p.ds_store) + (int64_t)b * p.ds_units * 8192;

  const int ent_lo = rec.ent_lo, n_ent = rec.n_ent;
  const int total = n_ent << cpb_sh;  // chunks
  EntryList list, units;
  list.init(p.q_tiles.ent + ent_lo, n_ent, lane);
  units.init(p.dq_units + ((int64_t)ent_lo << cpb_sh) * 2, total * 2, lane);
  // chunk j (clamped to the last one): its first key row and the unit that holds dS for my half of
  // the tile (-1: not mine)
  auto chunk_at = [&](int j, int& kv0, int& unit) S2_INLINE {
    const bool inside = j < total;
    j = min(j, total - 1);
    const int e = list.get(j >> cpb_sh, lane);
    kv0 = (e >> 16) * S + (j & cpb_m) * 64;
    unit = units.get(2 * j + qhalf, lane);
    if (!inside) unit = -1;
  };

  // K: the workgroup's 256 lanes fetch 16 rows x 16 pieces per load, this lane row 16 i + tid / 16 of
  // the chunk for load i, piece tid % 16; dS: my key half of the unit, 4 KiB in one run
  const int k_row = tid >> 4, k_piece = tid & 15;
  const int64_t k_goff = (int64_t)k_row * p.kv_st + 8 * k_piece;     // elements
  const int k_loff = k_row * Tile::kStride + 8 * k_piece;            // elements
  const uint32_t ds_goff = 4096 * khalf + lane * 16;                 // bytes
  struct Fetch {
    u32x4 k[4], ds[4];
  };
  auto fetch = [&](Fetch& f, int kv0, int unit) S2_INLINE {
    const uint16_t* kg = kb + (int64_t)kv0 * p.kv_st + k_goff;
#pragma unroll
    for (int i = 0; i < 4; ++i) f.k[i] = *reinterpret_cast<const u32x4*>(kg + (int64_t)(16 * i) * p.kv_st);
    // a chunk that is not mine fetches unit 0 (it exists) so that every step issues the same loads
    const unsigned char* ug = ds_b + (int64_t)max(unit, 0) * 8192 + ds_goff;
#pragma unroll
    for (int i = 0; i < 4; ++i) f.ds[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ug + 1024 * i));
  };
  // lane i of a run's kilobyte holds 16 bytes of key i / 4
  const uint32_t ds_loff = (lane >> 4) * kDsQuadStride + l16 * 16;
  auto stash = [&](const Fetch& f, int stage, int unit) S2_INLINE {
    uint16_t* kt = sm.loop.k[stage] + k_loff;
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(kt + 16 * i * Tile::kStride) = f.k[i];
    if (unit < 0) return;
    unsigned char* dw = sm.loop.ds[wave] + ds_loff;
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(dw + 4 * i * kDsQuadStride) = f.ds[i];
  };

  f32x4 acc[FT][4];  // dQ transposed [16-feature tile][16-query tile of my 64]
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int nq = 0; nq < 4; ++nq) acc[ft][nq] = f32x4{};
  const uint32_t tr_lane = lds_addr(sm.loop.k[0]) + Tile::tr_lane(lane) + Tile::tr_off(khalf, 0);
  // lane part of a dS transpose read: lane 4 e + q of group g supplies key 4 g + e, queries 4 q .. 4 q + 3 of a 16-query tile,
  // which lie in the key's 16 bytes of (the writer's) group q, the first or second eight of them by the tile's parity
  const uint32_t ds_lane = lds_addr(sm.loop.ds[wave]) + g * kDsQuadStride + (l16 >> 2) * 64 + (l16 & 3) * 16;

  auto multiply = [&](int kv0, int unit, int stage) S2_INLINE {
    if (unit < 0) return;
    // keys all after the first 32 queries: the dK/dV kernel skipped that quarter, nothing was stored
    // (the unit exists, so they are not after the second 32)
    const bool first = kv0 + 32 * khalf <= q0;
    bf16x8 ds[4];
#pragma unroll
    for (int nq = 0; nq < 4; ++nq) {
      // (the second four of the lane's keys are 16 keys further on)
      u32x4 r = lds_read_tr(ds_lane, (nq >> 1) * 8 * kDsQuadStride + 8 * (nq & 1), kDsQuadStride / 2);
      if (nq < 2 && !first) r = u32x4{0u, 0u, 0u, 0u};  // what LDS holds there is not dS: that quarter counts as zero
      ds[nq] = __builtin_bit_cast(bf16x8, r);
    }
    const uint32_t kt = tr_lane + stage * (uint32_t)Tile::kBytes;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) {
      const bf16x8 kf = __builtin_bit_cast(bf16x8, lds_read_tr(kt, Tile::tr_off(0, ft), 2 * Tile::RB));
#pragma unroll
      for (int nq = 0; nq < 4; ++nq) acc[ft][nq] = mfma16(kf, ds[nq], acc[ft][nq]);
    }
  };

  if (total > 0) {
    // chunks 0 and 1 requested, chunk 0 in LDS
    Fetch fa, fb;
    int kv0[3], unit[3];  // of chunks ch, ch + 1, ch + 2
    chunk_at(0, kv0[0], unit[0]);
    fetch(fa, kv0[0], unit[0]);
    chunk_at(1, kv0[1], unit[1]);
    fetch(fb, kv0[1], unit[1]);
    stash(fa, 0, unit[0]);
    __syncthreads();
    // Step ch: request chunk ch + 2 into the registers chunk ch came through, multiply chunk ch, move
    // chunk ch + 1 from its registers to LDS (the other K stage; my dS region after my own reads of
    // it, LDS serves a wavefront in order), barrier.  Two steps per trip so that the register sets
    // keep their names.
    for (int ch = 0; ch < total; ch += 2) {
      chunk_at(ch + 2, kv0[2], unit[2]);
      fetch(fa, kv0[2], unit[2]);
      multiply(kv0[0], unit[0], 0);
      stash(fb, 1, unit[1]);
      __syncthreads();
      if (ch + 1 >= total) break;
      chunk_at(ch + 3, kv0[0], unit[0]);
      fetch(fb, kv0[0], unit[0]);
      multiply(kv0[1], unit[1], 1);
      stash(fa, 0, unit[2]);
      __syncthreads();
      kv0[1] = kv0[0];
      unit[1] = unit[0];
      kv0[0] = kv0[2];
      unit[0] = unit[2];
    }
  }

  // The second key half hands its sums over through LDS (free since the loop's last barrier), register
  // by register with the lane as the fast index; the first adds them and owns the rows from here on.
  float* red = sm.reduce[qhalf] + lane;
  if (khalf == 1) {
#pragma unroll
    for (int ft = 0; ft < FT; ++ft)
#pragma unroll
      for (int nq = 0; nq < 4; ++nq)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((ft * 4 + nq) * 4 + r) * 64] = acc[ft][nq][r];
  }
  __syncthreads();
  if (khalf == 1) return;
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int nq = 0; nq < 4; ++nq)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[ft][nq][r] += red[((ft * 4 + nq) * 4 + r) * 64];

  // dQ = scale * acc goes out through LDS (my half of the reduction buffer, which only I read, after my
  // own reads of it), whole rows per store instruction
  constexpr int RS = D + 8;  // staging row stride (elements)
  uint16_t* stage = reinterpret_cast<uint16_t*>(sm.reduce[qhalf]);
  static_assert(64 * RS * 2 <= 64 * D * 4, "the staging rows fit the reduction buffer");
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int nq = 0; nq < 4; ++nq) {
      bf16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (__bf16)(acc[ft][nq][e] * p.scale);
      *reinterpret_cast<bf16x4*>(stage + (16 * nq + l16) * RS + 16 * ft + 4 * g) = w;
    }
  uint16_t* obase = p.dq + q_off + (int64_t)q0 * p.q_st;
#pragma unroll
  for (int i = 0; i < 64 / 4; ++i) {
    const int r = 4 * i + (lane >> 4), piece = lane & 15;
    const u32x4 x = *reinterpret_cast<const u32x4*>(stage + r * RS + 8 * piece);
    *reinterpret_cast<u32x4*>(obase + (int64_t)r * p.q_st + 8 * piece) = x;
  }
}

}  // namespace

hipError_t launch_dq_gemm(const AttnParams& p, hipStream_t stream) {
  static SmemSet set;  // zero-initialised
  const hipError_t e = set_smem(&dq_gemm_kernel<128>, sizeof(DqGemmSmem<128>), set);
  if (e != hipSuccess) return e;
  const int grid = (int)p.row_map.grid();
  hipLaunchKernelGGL((dq_gemm_kernel<128>), dim3(grid), dim3(kThreads), sizeof(DqGemmSmem<128>), stream, p);
  return hipGetLastError();
}

}  // namespace s2
