// Backward kernels: gradients of block-sparse causal attention (the backward pass that goes with
// the forward of section 3.2; the paper names it as the less optimised half of its kernels).
//
// Two launches (delta, then the tiles of dQ and dK/dV, in whole backwards of up to 4096 workgroups; dQ, then dK/dV, in larger ones; three
// where dS is kept: delta, dK/dV, dQ), no floating-point atomics, bitwise reproducible:
//   delta  : delta[t] = sum_d dO[t][d] * O[t][d].  Folded into the dq launch, which holds the dO
//            fragments anyway; the stand-alone kernel runs where dS is kept, where it is asked for without dQ, and
//            before the launch that does the tiles of both others (bwd_merged_kernel.hip).
//   dq     : row-stationary, in dq_pipe_kernel.hip (dq_gemm_kernel.hip where dS is kept).  A workgroup
//            owns 128 query rows and walks the merged list of KV blocks its mask rows keep (as the
//            forward does), recomputing P and forming dS = P * (dP - delta), dQ += scale * dS K.
//   dkdv   : column-stationary (dkdv_tile.h).  A workgroup owns 128 keys - one or two mask columns, paired by
//            the layout builder so that both are attended by nearly the same query blocks - and
//            walks the query blocks that keep them: dV += P^T dO, dK += scale * dS^T Q.  Where a launch
//            has few tiles, the longest are cut into parts for several workgroups; the last one to
//            finish adds the parts up in their order.  dK/dV launch of 2 x 16 heads x 4096 x 64 107 -> 56 us,
//            2 x 16 x 3904 x 128 163 -> 88, 1 x 16 x 8192 x 128 with 16-token blocks 355 -> 95.
//
// Both main kernels keep the stationary operand's MFMA fragments in registers with the lane
// owning one stationary row, so the recomputed score tile lands in the C layout with the
// streamed index in registers; it is then fed back as the B operand of the next contraction
// without leaving the lane (see device_util.h).  The streamed 64-row chunk is brought in by
// direct global -> LDS loads (double buffered) and read in both operand forms from the one
// row-major tile: row fragments (k = feature) and LDS transpose reads (k = token).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "config.h"
#include "device_util.h"
#include "dkdv_tile.h"
#include "kernels.h"
#include "smem_limit.h"

namespace s2 {

namespace {

// ------------------------------------------------------------------------------------ delta

// One pass over O and dO, bound by HBM.  A workgroup takes delta_rows<D>() rows of one head, four lanes to a row, a lane's 16-byte pieces
// 64 bytes apart and all its loads in flight together; one row to D / 8 lanes, each with a 64-bit division to find its head, took 57 us for 4 x 16 x
// 8192 x 128 and 109 for 1 x 32 x 32768 (4.7 and 4.9 TB/s).  The products are added up in the order of the dQ kernel, so that delta is
// the same to the bit wherever it is formed.
// VARLEN: a packed batch, whose tensors may hold many times the rows that are in use.  The grid has the rows that as many sequences
// of the longest length allowed would take; sequences that are cut at that length leave gaps, so the last row may lie beyond it
// and a workgroup goes on to the next such stretch.  What the last row is comes while the first stretch is being
// loaded.  8 sequences of 200 rows x 8 heads x 128 in tensors of 65536 rows, whole backward: 58 us with a pass over the whole tensors, 22 with this one.
template <int D>
constexpr int delta_rows() {
  return 64 * 128 / D;
}
template <int D>
int delta_tiles(const AttnParams& p) {  // a head's share of the grid
  const int64_t rows = p.cu_seqlens ? std::min<int64_t>(p.seqlen, (int64_t)p.batch * p.q_rows) : p.seqlen;
  return (int)((rows + delta_rows<D>() - 1) / delta_rows<D>());
}

// The end of the last row that belongs to a sequence, by the workgroup together.  lo, hi: row offsets of sequence tid (0 if there is none)
__device__ __forceinline__ int rows_in_use(const AttnParams& p, int tid, int lo, int hi) {
  __shared__ int ends[4];
  int end = 0;
  for (int b = tid;;) {
    const int row_base = min(max(lo, 0), p.seqlen);  // as the tiles read it
    end = max(end, row_base + min(min(max(hi - lo, 0), p.q_rows), p.seqlen - row_base));
    b += 256;
    if (b >= p.batch) break;
    lo = p.cu_seqlens[b];
    hi = p.cu_seqlens[b + 1];
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) end = max(end, __shfl_xor(end, m, 64));
  if ((tid & 63) == 0) ends[tid >> 6] = end;
  __syncthreads();
  return max(max(ends[0], ends[1]), max(ends[2], ends[3]));
}

template <int D, bool VARLEN>
__global__ __launch_bounds__(256) void delta_kernel(const AttnParams p, int tiles) {
  constexpr int KS = D / 32, ROWS = delta_rows<D>(), PASSES = ROWS / 64;
  const int tid = threadIdx.x, g = tid & 3;
  const int bh = blockIdx.x / tiles;
  const int b = bh / p.heads, h = bh - b * p.heads;  // (packed: b = 0)
  const int64_t base = b * p.q_sb + h * p.q_sh + 8 * g;
  int row0 = (blockIdx.x - bh * tiles) * ROWS, end = VARLEN ? -1 : p.seqlen;
  int lo = 0, hi = 0;
  if (VARLEN && tid < p.batch) {  // (asked for first, so that they are waited for alone)
    lo = p.cu_seqlens[tid];
    hi = p.cu_seqlens[tid + 1];
  }
  do {
    const int t0 = row0 + (tid >> 2);
    bf16x8 o[PASSES][KS], d[PASSES][KS];
    float lse[PASSES];
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      // (a row past the end reads the last one; nothing of it is stored)
      const int t = min(t0 + 64 * i, p.seqlen - 1);
      const int64_t off = base + t * p.q_st;
      lse[i] = p.lse[(int64_t)bh * p.seqlen + t];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        o[i][kk] = *reinterpret_cast<const bf16x8*>(p.o + off + 32 * kk);
        d[i][kk] = *reinterpret_cast<const bf16x8*>(p.d_o + off + 32 * kk);
      }
    }
    if (VARLEN) {
      if (end < 0) end = rows_in_use(p, tid, lo, hi);
      if (row0 >= end) return;
    } else {
      clear_split_counts(p, blockIdx.x * 256 + tid);  // (a packed batch has no tiles that are cut)
    }
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      float acc = 0.f;
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = __builtin_fmaf((float)d[i][kk][e], (float)o[i][kk][e], acc);
      // (without the LDS; with lse on its way from the start 1 x 5 x 4096 x 64 backward 27.8 -> 27.1 us, 1 x 4 x 512 15.8 -> 15.5)
      acc += dpp<0x4E>(acc);  // quad_perm 2301: of lane ^ 2
      acc += dpp<0xB1>(acc);  // quad_perm 1032: of lane ^ 1
      const int t = t0 + 64 * i;
      if (g == 0 && t < end) {
        const int64_t row = (int64_t)bh * p.seqlen + t;
        p.neg_delta[row] = -acc;
        p.neg_lse[row] = lse[i] * p.neg_inv_scale;
      }
    }
    row0 += tiles * ROWS;
  } while (VARLEN && row0 < end);
}

template <int D, bool DENSE, int FINE, bool VARLEN, bool STORE>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 3) void dkdv_kernel(const AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  dkdv_tile<D, DENSE, FINE, VARLEN, STORE>(p, blockIdx.x, smem_raw);
}

template <int D, bool DENSE, int FINE, bool VARLEN, bool STORE>
hipError_t launch_dkdv(const AttnParams& p, hipStream_t stream) {
  static SmemSet set;  // zero-initialised
  hipError_t e = set_smem(&dkdv_kernel<D, DENSE, FINE, VARLEN, STORE>, sizeof(DkvSmem<D>), set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((dkdv_kernel<D, DENSE, FINE, VARLEN, STORE>), dim3(p.key_map.grid()),
                     dim3(kThreads), sizeof(DkvSmem<D>), stream, p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_delta(const AttnParams& p, hipStream_t stream) {
  const int tiles = delta_tiles<D>(p);
  // (a packed batch: one run of rows a head)
  if (p.cu_seqlens)
    hipLaunchKernelGGL((delta_kernel<D, true>), dim3((unsigned)p.heads * tiles), dim3(256), 0, stream, p, tiles);
  else
    hipLaunchKernelGGL((delta_kernel<D, false>), dim3((unsigned)((int64_t)p.batch * p.heads * tiles)), dim3(256), 0, stream, p, tiles);
  return hipGetLastError();
}

// For a dK/dV launch that is not preceded by delta or dQ in its own call, which brings delta from an earlier one and nothing else: -lse /
// scale goes by this call's scale, and what is in the counters of the cut key tiles is not known (the earlier call may
// have had a smaller workspace).
__global__ __launch_bounds__(256) void prepare_dkdv_kernel(const AttnParams p) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (more rows than tiles)
  clear_split_counts(p, (int)min(i, (int64_t)1 << 30));
  if (i < (int64_t)p.batch * p.heads * p.seqlen) p.neg_lse[i] = p.lse[i] * p.neg_inv_scale;
}

hipError_t launch_prepare_dkdv(const AttnParams& p, hipStream_t stream) {
  const int64_t rows = (int64_t)p.batch * p.heads * p.seqlen;
  hipLaunchKernelGGL(prepare_dkdv_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_dim(const AttnParams& p, bool dense, int stages, hipStream_t stream) {
  hipError_t e = hipSuccess;
  if constexpr (D == 128) {
    if (p.ds_store) {
      // The backward that keeps dS: delta, then dK/dV (5 contractions' worth of work less the dQ one,
      // leaving dS in the workspace), then dQ = scale * dS K - nothing is computed twice.
      if (stages & kBwdDelta)
        e = launch_delta<D>(p, stream);
      else if (stages & kBwdDkDv)
        e = launch_prepare_dkdv(p, stream);
      if (e == hipSuccess && (stages & kBwdDkDv)) e = launch_dkdv<D, false, 0, false, true>(p, stream);
      if (e == hipSuccess && (stages & kBwdDq)) e = launch_dq_gemm(p, stream);
      return e;
    }
  }
  // (a call for some of the stages keeps the launches that it names)
  if ((stages & kBwdAll) == kBwdAll && bwd_is_merged(p)) {
    e = launch_delta<D>(p, stream);
    return e == hipSuccess ? launch_bwd_merged(p, dense, stream) : e;
  }
  // The dQ kernel computes delta itself and leaves the row statistics in the workspace,
  // so it runs first, and of the other two launches the stand-alone delta kernel only when dQ is not part of the call
  // (a packed batch is always a whole backward).
  if (stages & kBwdDq)
    e = launch_dq(p, dense, stream);
  else if (stages & kBwdDelta)
    e = launch_delta<D>(p, stream);
  else
    e = launch_prepare_dkdv(p, stream);
  if (e != hipSuccess || !(stages & kBwdDkDv)) return e;
  if (dense) return launch_dkdv<D, true, 0, false, false>(p, stream);
  if (p.cu_seqlens) {
    if (p.block_size == 16) return launch_dkdv<D, false, 16, true, false>(p, stream);
    if (p.block_size == 32) return launch_dkdv<D, false, 32, true, false>(p, stream);
    return launch_dkdv<D, false, 0, true, false>(p, stream);
  }
  if (p.block_size == 16) return launch_dkdv<D, false, 16, false, false>(p, stream);
  if (p.block_size == 32) return launch_dkdv<D, false, 32, false, false>(p, stream);
  return launch_dkdv<D, false, 0, false, false>(p, stream);
}

}  // namespace

hipError_t launch_bwd(const AttnParams& params, bool dense, int stages, hipStream_t stream) {
  AttnParams p = params;
  const int pairs = p.batch * p.heads, tiles = (p.q_rows + kBwdBM - 1) / kBwdBM;
  p.row_map = row_map(pairs, tiles, map_group(pairs, tiles, p.cu_seqlens != nullptr), dense ? kDenseRows : kSparseRows, xcd_slots(p.head_dim));
  p.key_map = key_map(pairs, p.kv_tiles.tiles_per_head + p.split_items - p.split_long);
  p.by_heads = fast_div(p.heads);
  return p.head_dim == 128 ? launch_dim<128>(p, dense, stages, stream) : launch_dim<64>(p, dense, stages, stream);
}

}  // namespace s2
