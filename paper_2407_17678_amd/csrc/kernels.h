// Internal: parameter blocks and launch entry points of the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "config.h"
#include "tile_map.h"

namespace s2 {

// A word, or a few, that no kernel writes, at an address that is the same for the whole wavefront: a scalar load.  (Where a kernel has stored
// something before, the compiler itself takes a vector load and waits for it.)
template <class T>
__device__ __forceinline__ T load_const(const void* p) {
  return *reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}

// Merged tile list on the device (see TileList in layout.h).
struct DevTiles {
  const int32_t* ptr = nullptr;
  const int32_t* ent = nullptr;
  const int32_t* rec = nullptr;  // [head][rank][kRowRec or kColRec]
  int tiles_per_head = 0;
  int group = 0;
  // What the workgroup of head h's tile of a rank begins with (layout.h: TileList::rec).
  // (The empty assembly has a row tile's words loaded together: left alone the compiler asks for each when it needs it.)
  struct RowRec {
    int tile, ent_lo, n_ent;
  };
  __device__ __forceinline__ RowRec row_rec(int h, int rank) const {
    typedef int32_t words __attribute__((ext_vector_type(4)));
    const words w = load_const<words>(rec + ((int64_t)h * tiles_per_head + rank) * kRowRec);
    RowRec r{w[0], w[1], w[2]};
    asm volatile("" : "+s"(r.tile), "+s"(r.ent_lo), "+s"(r.n_ent));
    return r;
  }
  __device__ __forceinline__ const int32_t* col_rec(int h, int rank) const { return rec + ((int64_t)h * tiles_per_head + rank) * kColRec; }
};

struct AttnParams {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* o;
  float* lse;
  const uint16_t* d_o;
  uint16_t* dq;
  uint16_t* dk;
  uint16_t* dv;
  // Workspace, [batch, heads, seqlen] each: what the dK/dV kernel's accumulators begin with, so that the score contraction ends
  // at S - lse / scale (P = exp2 of it times p_scale_log2e) and the other at dP - delta
  float* neg_delta;  // -rowsum(dO * O)
  float* neg_lse;    // lse * neg_inv_scale
  int batch, heads, seqlen, head_dim;
  // q, o, lse hold q_rows rows, local row r being sequence position q_row0 + r (the whole sequence,
  // as in every backward of a fixed length: q_row0 = 0, q_rows = seqlen)
  int q_row0, q_rows;
  // packed variable-length batch (nullptr = every sequence has seqlen rows):
  // sequence b owns rows cu_seqlens[b] .. cu_seqlens[b+1]-1 of q, k, v, o and lse; then batch is
  // the number of sequences, seqlen the rows in the tensors and q_rows the longest length allowed
  const int32_t* cu_seqlens;
  // which tile a workgroup computes (tile_map.h; set by launch_fwd and launch_bwd)
  RowMap row_map;
  KeyMap key_map;
  FastDiv by_heads;
  int64_t q_sb, q_sh, q_st;
  int64_t kv_sb, kv_sh, kv_st;
  float scale;        // softmax scale
  float scale_log2e;  // scale * log2(e)
  // Backward: the scale of the dK/dV kernel's exponent is the softmax scale or, if that is smaller, 2^-120 (make_params)
  float neg_inv_scale;  // -1 / that
  float p_scale_log2e;  // that * log2(e)
  int block_size;     // S (sparse path); 64 on the dense path
  DevTiles q_tiles;   // row tiles of the forward and dQ kernels -> KV blocks
  DevTiles kv_tiles;  // column tiles -> Q blocks
  // Key tiles cut into parts (SplitLevel in layout.h; split_items == 0: none are): the first split_items
  // items of a head are parts of its first split_long tiles.  The parts' sums go to split_sums, [batch *
  // heads][item][wavefront][accumulator quad][lane][4] floats, and split_count[batch * heads][tile] counts the
  // parts that are done: it is zero before the launch (the launch before it clears it: the one that leaves delta, or the
  // one that prepares a call for dK/dV alone).
  const int32_t* split_codes;
  float* split_sums;
  int32_t* split_count;
  int split_items, split_long;
  // Backward with dS kept (head_dim 128, mask blocks of 64 or 128 tokens): the dK/dV kernel leaves
  // dS = P * (dP - delta), rounded to bf16, in the workspace, in units of 64 queries x 64 keys (8 KiB),
  // unit (2 * step + wavefront pair) of its walk; the dQ launch is then the one contraction dS K over
  // those units.  ds_store == nullptr: dS is not kept and the dQ kernel recomputes it.
  uint16_t* ds_store;          // [batch][ds_units] units
  int64_t ds_units;            // units per batch element
  const int32_t* dq_units;     // [dQ list chunk][query half of the 128-row tile]: unit, -1 = none
};

// Clears the counters of the key tiles that are cut, thread i of a launch that precedes the dK/dV launch
// (it has at least as many threads as there are tiles).
__device__ __forceinline__ void clear_split_counts(const AttnParams& p, int i) {
  if (p.split_items > 0 && i < p.batch * p.heads * p.kv_tiles.tiles_per_head) p.split_count[i] = 0;
}

struct DecodeParams {
  const uint16_t* q;
  const uint16_t* k_cache;
  const uint16_t* v_cache;
  const int32_t* seq_lens;
  uint16_t* o;
  float* lse;
  float* part_acc;  // [nseq*heads*splits, head_dim]
  float* part_ml;   // [nseq*heads*splits, 2]  (max, sum)
  int nseq, heads, head_dim, max_len, num_splits;
  int64_t kv_ss, kv_sh, kv_st;
  float scale, scale_log2e;
  int block_size, local_blocks, stride, window_blocks, dense, head_index_base;
  // paged cache: k_cache / v_cache are the page pools, kv_ss is the page stride
  const int32_t* block_table;  // [nseq, heads, max_blocks], nullptr = contiguous cache
  int32_t* missing;            // optional counter of kept blocks that are not resident
  int max_blocks, num_pages;
  // caller-supplied pattern: the kept blocks of row i of head h are
  // col_idx[row_ptr[h*num_blocks + i] .. row_ptr[h*num_blocks + i + 1]); nullptr = closed form
  const int32_t* row_ptr;
  const int32_t* col_idx;
  int num_blocks;
  FastDiv by_heads, by_splits, by_stride;  // set by launch_decode
};

// Each returns the hipError_t of the launch (hipGetLastError after the launch).
hipError_t launch_fwd(const AttnParams& p, bool dense, hipStream_t stream);
// The launch of it for mask blocks of 16 and 32 tokens (row_map set).
hipError_t launch_fwd_gather(const AttnParams& p, hipStream_t stream);
// `stages` selects which of the three backward launches run: 1 = delta, 2 = dK/dV, 4 = dQ.
constexpr int kBwdDelta = 1, kBwdDkDv = 2, kBwdDq = 4, kBwdAll = 7;
hipError_t launch_bwd(const AttnParams& p, bool dense, int stages, hipStream_t stream);
// The dQ launch that recomputes S and dP (it also leaves the row statistics in the workspace).
hipError_t launch_dq(const AttnParams& p, bool dense, hipStream_t stream);
// The dQ launch of the backward that keeps dS: dQ = scale * dS K over the stored units.
hipError_t launch_dq_gemm(const AttnParams& p, hipStream_t stream);
// dQ and dK/dV of a backward that recomputes S and dP in one launch, after delta: whether the two are better off so, and the launch.
bool bwd_is_merged(const AttnParams& p);
hipError_t launch_bwd_merged(const AttnParams& p, bool dense, hipStream_t stream);
// The most workgroups of a decode call that are of eight wavefronts instead of four.  One to a compute unit, they
// keep twice the units of a (sequence, head) in flight: 32 pairs of 16 units in one split 13.2 -> 9.8 us, 224 pairs of
// 4096 to 8192 tokens, 64-token blocks, 8 local + stride 8, D = 64, 15.9 -> 15.7, with 32-token blocks (16 + stride 16)
// 15.2 -> 12.9.  Once there are two to a compute unit four are enough, and end more evenly (288 pairs, 64-token blocks,
// 16 + stride 16, 32768 tokens, D = 64: 38.8 and, with eight, 41.0), except that with 16-token blocks at D = 64, whose
// units are the smallest, eight stay ahead in long rows up to 512 (288 pairs of 8192 tokens 13.4 -> 12.6, 512 pairs
// 17.5 -> 17.2; rows of 2048 tokens 5.7 and 5.8).
constexpr int kDecodeWideGroups = 256;
constexpr int decode_wide_groups(int block_size, int head_dim) {
  return block_size == 16 && head_dim == 64 ? 2 * kDecodeWideGroups : kDecodeWideGroups;
}
hipError_t launch_decode(const DecodeParams& p, hipStream_t stream);

}  // namespace s2
