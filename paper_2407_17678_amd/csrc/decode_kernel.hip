// Decode: one query token per sequence against a contiguous KV cache (section 4.1).  The query
// at position L-1 reads only the KV blocks that block row (L-1) div S of the head's mask keeps:
// the head's vertical stripes plus the local window (section 4.2), enumerated in closed form.
// The work is one multiply-add per byte read, so the kernel is a bandwidth kernel in large calls and a chain of latencies
// in small ones: every lane issues 16-byte loads, a row of K or V is covered by D/8 adjacent lanes, and a wavefront always
// has a K or V tile of 64 tokens on its way: the next unit's K is requested as soon as this unit's scores have freed
// the registers, its V as soon as the sums have.  What is the same in all lanes (the list entry, the page, the block's
// address, the rows attended) is found by scalar instructions, a unit ahead, and counted once: a block is a
// buffer that ends with its last attended row, so that a load needs no clamping (a row past the end reads as
// zero and fetches nothing) and its address is one scalar addition.  Scores are added up across a row's lanes by lane
// permutations inside the additions; through the LDS each took four round trips that a lone wavefront waits for.  Measured
// against one lookup per lane and load, loads of a unit behind the sums of the one before and sums through the LDS: 40 x 30 paged
// rows of 4000 to 16384 x 64, blocks of 16 87 -> 70 us, 64 x 32 paged rows of 8192 to 32768 x 128 (blocks of 16) 258 -> 238
// (5.8 TB/s), 224 rows of 4096 to 8192, D = 64, blocks of 64 17.5 -> 14.0, one sequence of 32768 x 32 heads with its merge 14.6 -> 13.3,
// calls of a few short rows 6.3 -> 4.6; 64 x 32 contiguous rows of 8192 to 16384 x 128 308 -> 305 (the same).
//
// A caller-supplied pattern replaces the closed form by row (L-1) div S of the layout's lists.
//
// Paged cache (PAGED = true): a kept block's rows are found through the block table instead of
// by offset into a contiguous cache; nothing else changes, since a page is one contiguous block.
//
// Split-KV: the list of 64-token units of one (sequence, head) is cut into num_splits pieces, one
// workgroup each; the four or eight wavefronts of a workgroup take units round-robin and merge their
// (max, sum, accumulator) through LDS; a second kernel merges the splits.  With one split per
// (sequence, head) the first kernel writes the result itself and the second is not launched.
#include <hip/hip_runtime.h>

#include "config.h"
#include "device_util.h"
#include "kernels.h"
#include "sched_util.h"

namespace s2 {

namespace {

constexpr float kNegInf = -__builtin_inff();

// From this token stride (in elements) on, the offsets of a unit's 64 rows do not fit into the 31 bits of a buffer's size.
constexpr int64_t kFarRows = (int64_t)1 << 24;

// Kept blocks of block row i, in ascending order, as (stripe run, local run), or as a list.
struct RowBlocks {
  int first_stripe, n_stripe, stride, local_lo, count;
  const int32_t* cols;  // caller-supplied pattern: the row's list; nullptr = closed form
  __device__ int block(int n) const {
    const int striped = first_stripe + n * stride, local = local_lo + (n - n_stripe);
    if (cols) return load_const<int32_t>(cols + n);
    return n < n_stripe ? striped : local;
  }
};

__device__ inline RowBlocks row_blocks(const DecodeParams& p, int head, int i) {
  RowBlocks r;
  r.stride = p.stride;
  r.first_stripe = 0;
  r.n_stripe = 0;
  r.cols = nullptr;
  r.local_lo = 0;
  if (p.row_ptr) {
    const int32_t lo = load_const<int32_t>(p.row_ptr + (int64_t)head * p.num_blocks + i);
    r.cols = p.col_idx + lo;
    r.count = load_const<int32_t>(p.row_ptr + (int64_t)head * p.num_blocks + i + 1) - lo;
    return r;
  }
  if (p.dense) {
    r.local_lo = 0;
    r.count = i + 1;
    return r;
  }
  r.local_lo = max(0, i - p.local_blocks + 1);
  if (p.stride > 0) {
    const int o = p.head_index_base + head - (p.head_index_base + head) / p.by_stride * p.stride;
    const int lo = p.window_blocks > 0 ? max(0, i - p.window_blocks + 1) : 0;
    int first = o;
    if (lo > o) first = o + (lo - o + p.stride - 1) / p.by_stride * p.stride;
    if (first < r.local_lo) {
      r.first_stripe = first;
      r.n_stripe = (r.local_lo - 1 - first) / p.by_stride + 1;
    }
  }
  r.count = r.n_stripe + (i - r.local_lo + 1);
  return r;
}

// GATHER: the instantiation for 16-token blocks, where a unit of work is four consecutive kept blocks
// of the row's list side by side, so that every load still fetches rows the query attends (a 16-token
// block on its own would fill a quarter of the 64 rows a unit loads).
//
// W: wavefronts of a workgroup, each with a unit in flight (128 data registers at D = 128, so two to a SIMD; three, with the
// registers pressed to 168, measured the same).
//
// FAR: the instantiation for caches whose tokens are so far apart that a unit does not fit a buffer's 31 bits (kFarRows): it
// reads through 64-bit addresses, and a row past the last attended one reads that one.
template <int D, bool PAGED, bool GATHER, int W, bool FAR>
__global__ __launch_bounds__(64 * W, FAR ? 1 : D == 128 ? 2 : 4) void decode_split_kernel(const DecodeParams p) {
  constexpr int LPR = D / 8;     // lanes covering one row
  constexpr int RPI = 64 / LPR;  // rows covered by one wavefront-wide load
  constexpr int NI = 64 / RPI;   // loads per 64-token unit

  __shared__ float sh_m[W], sh_l[W];
  __shared__ float sh_acc[W][D];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (a unit's blocks and pages are then found by scalar instructions)
  const int c = lane % LPR, g = lane / LPR;
  const int item = blockIdx.x;  // (b * heads + h) * splits + split
  const int bh = item / p.by_splits, split = item - bh * p.num_splits;
  const int b = bh / p.by_heads, h = bh - b * p.heads;

  int L = load_const<int32_t>(p.seq_lens + b);
  L = min(max(L, 1), p.max_len);
  const int32_t* table = PAGED ? p.block_table + ((int64_t)b * p.heads + h) * p.max_blocks : nullptr;
  const int S = p.block_size;
  const int U = min(S, kChunk);  // tokens per unit of work: 64, or a whole block when it is shorter
  const int cpb_sh = S == 128 ? 1 : 0, cpb = 1 << cpb_sh;  // units of a block
  constexpr int BPU = 4;         // GATHER: blocks per unit
  const int i = (L - 1) >> (31 - __builtin_clz(S));
  const RowBlocks rb = row_blocks(p, h, i);
  const int units = GATHER ? (rb.count + BPU - 1) / BPU : rb.count << cpb_sh;
  // units * split / num_splits and units * (split + 1) / num_splits, without 64-bit divisions
  const int even = units / p.by_splits, rest = units - even * p.num_splits;
  const int u_lo = even * split + rest * split / p.by_splits, u_hi = even * (split + 1) + rest * (split + 1) / p.by_splits;

  // my 8 query features, as floats
  float qv[8];
  {
    const bf16x8 q8 = *reinterpret_cast<const bf16x8*>(p.q + ((int64_t)b * p.heads + h) * D + 8 * c);
#pragma unroll
    for (int e = 0; e < 8; ++e) qv[e] = (float)q8[e];
  }
  const uint16_t* kb = p.k_cache + (PAGED ? 0 : b * p.kv_ss + h * p.kv_sh);
  const uint16_t* vb = p.v_cache + (PAGED ? 0 : b * p.kv_ss + h * p.kv_sh);
  int n_missing = 0;
  const float cl = p.scale_log2e;

  float m_run = kNegInf, l_run = 0.f;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;

  // A unit is 64 rows: NB blocks of 16 (GATHER), else a run of rows of one block.
  constexpr int NB = GATHER ? BPU : 1, NPB = NI / NB;  // loads to a block
  struct Unit {
    int64_t base[NB];  // element offset of the block's first row of the unit
    int rows[NB];      // how many of its rows the query attends (GATHER: none of a block past the list's end, past L or not there)
  };
  auto unit_at = [&](int u) {
    Unit w;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int bi = GATHER ? u * BPU + i : u >> cpb_sh;
      const bool inside = !GATHER || bi < rb.count;
      const int blk = rb.block(inside ? bi : 0);
      const int skip = GATHER ? 0 : (u & (cpb - 1)) * U;  // rows of the block before the unit's
      const int tok0 = blk * S + skip;
      w.rows[i] = inside ? min(L - tok0, U) : 0;
      w.base[i] = FAR ? tok0 * p.kv_st : (int64_t)((uint64_t)(uint32_t)tok0 * (uint32_t)p.kv_st);
      if (PAGED) {
        const int page = load_const<int32_t>(table + blk);
        const bool resident = page >= 0 && page < p.num_pages;
        // kept by the mask but not there: counted, for a block of several units with the first
        if (inside && !resident) {
          n_missing += skip == 0;
          w.rows[i] = 0;
        }
        w.base[i] = (int64_t)((uint64_t)(uint32_t)page * (uint64_t)p.kv_ss) + skip * p.kv_st;
      }
    }
    return w;
  };
  // the first of the units u, u + W, ... before u_hi that has a row to read (GATHER: the unit u); u is moved there
  auto find = [&](int& u) {
    Unit w{};
    for (; u < u_hi; u += W) {
      w = unit_at(u);
      if (GATHER || w.rows[0] > 0) break;  // else the second half of a partial last block, or a block that is not resident
    }
    return w;
  };
  const uint32_t mine = 2 * (g * (uint32_t)p.kv_st + 8 * c), step = 2 * RPI * (uint32_t)p.kv_st;
  auto load = [&](const uint16_t* from, const Unit& w, bf16x8 (&x)[NI]) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const uint16_t* at = from + w.base[i];
      if constexpr (FAR) {
        // (a row past the last one attended reads that one; a block without one is zeros, as from an empty buffer: its weights
        // are 0, and 0 times what lies in a page that nobody owns need not be)
        const int last = w.rows[i] - 1;
#pragma unroll
        for (int n = 0; n < NPB; ++n)
          x[NPB * i + n] = last < 0 ? bf16x8{} : *reinterpret_cast<const bf16x8*>(at + (int64_t)min(RPI * n + g, last) * p.kv_st + 8 * c);
      } else {
        const auto rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(at), 0, max(w.rows[i], 0) * (int)(2 * p.kv_st), 0x00020000);
#pragma unroll
        for (int n = 0; n < NPB; ++n)
          x[NPB * i + n] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rows, mine + n * step, 0, 0));
      }
    }
  };

  bf16x8 kr[NI], vr[NI];
  float s[NI], mx;
  auto scores = [&](const Unit& w) __attribute__((always_inline)) {
    mx = kNegInf;
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      float d = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) d = __builtin_fmaf(qv[e], (float)kr[n][e], d);
      d += of_neighbour<1>(d);
      d += of_neighbour<2>(d);
      d += of_neighbour<4>(d);
      if (LPR == 16) d += of_neighbour<8>(d);
      if (RPI * (n % NPB) + g >= w.rows[n / NPB]) d = kNegInf;
      s[n] = d;
      mx = fmaxf(mx, d);
    }
  };
  auto sums = [&]() __attribute__((always_inline)) {
    if (LPR == 8) mx = fmaxf(mx, of_neighbour<8>(mx));
    mx = max_halves(max_rows(mx));
    const float m_new = fmaxf(m_run, mx);
    // (GATHER: nothing live yet in a paged cache with the unit's blocks missing, every weight is 0; else the unit's first
    // token is attended)
    const bool live = !GATHER || m_new != kNegInf;
    const float alpha = fast_exp2(live ? (m_run - m_new) * cl : 0.f);
    const float mc = live ? m_new * cl : 0.f;
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= alpha;
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      const float pr = fast_exp2(__builtin_fmaf(s[n], cl, -mc));
      psum += pr;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(pr, (float)vr[n][e], acc[e]);
    }
    l_run = l_run * alpha + psum;  // per row group; groups are summed at the end
    m_run = m_new;
  };

  int u = u_lo + wave;
  Unit w = find(u);
  if (u < u_hi) {
    load(kb, w, kr);
    load(vb, w, vr);
    for (;;) {
      u += W;
      const Unit next = find(u);
      if (u >= u_hi) break;
      // the next unit's K goes into the registers that the scores have freed, its V into those that the sums free
      scores(w);
      __builtin_amdgcn_sched_barrier(0);  // (the compiler mixes the loads into the sums otherwise, and waits for the last of them)
      load(kb, next, kr);
      __builtin_amdgcn_sched_barrier(0);
      sums();
      __builtin_amdgcn_sched_barrier(0);
      load(vb, next, vr);
      w = next;
    }
    scores(w);
    sums();
  }

  if (PAGED && p.missing && lane == 0 && n_missing > 0) atomicAdd(p.missing, n_missing);

  // sum the row groups of the wavefront
  if (LPR == 8) l_run += of_neighbour<8>(l_run);
  l_run = sum_halves(sum_rows(l_run));
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (LPR == 8) acc[e] += __shfl_xor(acc[e], 8, 64);  // (other features in each lane of a group)
    acc[e] = sum_halves(sum_rows(acc[e]));
  }
  if (lane == 0) {
    sh_m[wave] = m_run;
    sh_l[wave] = l_run;
  }
  if (g == 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) sh_acc[wave][8 * c + e] = acc[e];
  }
  __syncthreads();
  if (tid < D) {
    float m = sh_m[0];
#pragma unroll
    for (int w = 1; w < W; ++w) m = fmaxf(m, sh_m[w]);
    float l = 0.f, a = 0.f;
    if (m > kNegInf) {
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float wgt = fast_exp2((sh_m[w] - m) * cl);  // exp2(-inf) = 0 for an idle wavefront
        l += sh_l[w] * wgt;
        a += sh_acc[w][tid] * wgt;
      }
    }
    if (p.num_splits == 1) {
      // the only split of its (sequence, head): the result itself, no partials and no second kernel
      // (l == 0 only when nothing was attended: a paged cache with every kept block missing)
      const __bf16 out = (__bf16)(l > 0.f ? a / l : 0.f);
      p.o[(int64_t)bh * D + tid] = *reinterpret_cast<const uint16_t*>(&out);
      if (tid == 0 && p.lse) p.lse[bh] = l > 0.f ? m * p.scale + __logf(l) : kNegInf;
      return;
    }
    p.part_acc[(int64_t)item * D + tid] = a;
    if (tid == 0) {
      p.part_ml[(int64_t)item * 2 + 0] = m;
      p.part_ml[(int64_t)item * 2 + 1] = l;
    }
  }
}

// Merges the splits of one (sequence, head).  What it costs is latency (a launch of few bytes), so the first
// partials are requested together with the (max, sum) pairs, one split to a lane, and groups of D / 4 lanes
// each add up the splits of their own.  The pairs are merged by lane permutations: twelve round trips through the LDS before
// (one sequence of 32768 x 32 heads, both launches, 13.9 -> 13.5 us).
template <int D>
__global__ __launch_bounds__(256) void decode_reduce_kernel(const DecodeParams p) {
  constexpr int LPR = D / 4;      // lanes covering one partial
  constexpr int NG = 256 / LPR;   // partials covered by the workgroup at a time
  constexpr int NP = 4;           // partials a group requests at a time
  __shared__ f32x4 sh[NG][LPR];
  const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int g = tid / LPR, c = tid % LPR, n = p.num_splits;
  const f32x4* part = reinterpret_cast<const f32x4*>(p.part_acc) + (int64_t)bh * n * LPR + c;
  const float* ml = p.part_ml + (int64_t)bh * n * 2;
  f32x4 x[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) x[i] = part[(int64_t)min(g + NG * i, n - 1) * LPR];
  const float ms = lane < n ? ml[2 * lane] : kNegInf;
  const float ls = lane < n ? ml[2 * lane + 1] : 0.f;
  float m = ms;
  m = fmaxf(m, of_neighbour<1>(m));
  m = fmaxf(m, of_neighbour<2>(m));
  m = fmaxf(m, of_neighbour<4>(m));
  m = max_halves(max_rows(fmaxf(m, of_neighbour<8>(m))));
  // (an empty split weighs nothing)
  const float wgt = ms == kNegInf ? 0.f : fast_exp2((ms - m) * p.scale_log2e);
  float l = ls * wgt;
  l += of_neighbour<1>(l);
  l += of_neighbour<2>(l);
  l += of_neighbour<4>(l);
  l += of_neighbour<8>(l);
  l = sum_halves(sum_rows(l));
  f32x4 a = f32x4{};
  for (int s0 = 0;;) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int s = s0 + g + NG * i;
      const float w = __shfl(wgt, s & 63, 64);
      if (s < n) a += x[i] * w;
    }
    s0 += NG * NP;
    if (s0 >= n) break;
#pragma unroll
    for (int i = 0; i < NP; ++i) x[i] = part[(int64_t)min(s0 + g + NG * i, n - 1) * LPR];
  }
  sh[g][c] = a;
  __syncthreads();
  if (tid >= LPR) return;
#pragma unroll
  for (int i = 1; i < NG; ++i) a += sh[i][c];
  // l == 0 only when nothing was attended: a paged cache with every kept block missing
  bf16x4 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) out[e] = (__bf16)(l > 0.f ? a[e] / l : 0.f);
  *reinterpret_cast<bf16x4*>(p.o + (int64_t)bh * D + 4 * c) = out;
  if (tid == 0 && p.lse) p.lse[bh] = l > 0.f ? m * p.scale + __logf(l) : kNegInf;
}

template <int D, int W, bool FAR>
void launch_split(const DecodeParams& p, hipStream_t stream) {
  const dim3 grid(p.nseq * p.heads * p.num_splits), block(64 * W);
  if (p.block_size == 16) {
    if (p.block_table)
      hipLaunchKernelGGL((decode_split_kernel<D, true, true, W, FAR>), grid, block, 0, stream, p);
    else
      hipLaunchKernelGGL((decode_split_kernel<D, false, true, W, FAR>), grid, block, 0, stream, p);
  } else if (p.block_table) {
    hipLaunchKernelGGL((decode_split_kernel<D, true, false, W, FAR>), grid, block, 0, stream, p);
  } else {
    hipLaunchKernelGGL((decode_split_kernel<D, false, false, W, FAR>), grid, block, 0, stream, p);
  }
}

template <int D>
hipError_t launch_one(const DecodeParams& p, hipStream_t stream) {
  const int bh = p.nseq * p.heads;
  if (p.kv_st >= kFarRows)
    launch_split<D, 4, true>(p, stream);
  else if (bh * p.num_splits <= decode_wide_groups(p.block_size, D))
    launch_split<D, 8, false>(p, stream);
  else
    launch_split<D, 4, false>(p, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.num_splits == 1) return e;  // a single split writes the result itself
  hipLaunchKernelGGL((decode_reduce_kernel<D>), dim3(bh), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_decode(const DecodeParams& params, hipStream_t stream) {
  DecodeParams p = params;
  p.by_heads = fast_div(p.heads);
  p.by_splits = fast_div(p.num_splits);
  p.by_stride = fast_div(p.stride > 0 ? p.stride : 1);
  return p.head_dim == 128 ? launch_one<128>(p, stream) : launch_one<64>(p, stream);
}

}  // namespace s2
