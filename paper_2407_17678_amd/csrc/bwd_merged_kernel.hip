// The backward's dQ tiles and dK/dV tiles in one launch, where each of the two launches would leave much of the chip idle, or idle at its end:
// dK/dV waits for nothing of dQ but delta, which the stand-alone kernel then forms first (to the same bits).  The tiles are those of the
// two kernels and so are the results, bit for bit.  Forward and backward, in two launches and in delta and one:
//   workgroups in all   head_dim 64                                        head_dim 128
//      64    1 x  4 x   512: 35.7 and  27.1 us                            47.0 and  33.5 us
//     256    1 x  8 x  2048: 48.8 and  37.6                               65.0 and  49.9
//    1024    2 x 16 x  2048: 62.5 and  56.3, dense 124.7 and 115.6       122.2 and 103.7, dense 193.3 and 172.2
//    2048    2 x 16 x  4096: 117  and 110;   dense 330   and 331         162   and 157 (4 x 16 x 2048); dense 568 and 545
//    4096    4 x 16 x  4096: 209  and 208;   packed 108  and  94         388   and 386;                 packed 161 and 156
//            dense 32 x 8192: 1149 and 1142; 128 x 2048: 342 and 346     dense 1969 and 1972;           602 and 606
//    6144    packed          141  and 125                                216   and 215
//    8192    8 x 16 x  4096: 411  and 413;   packed 174  and 158         748   and 761;                 packed 283 and 281
//            16-token        366  and 366;   packed 183  and 167         683   and 696;                 packed 297 and 295
//   16384    packed          274  and 277                                513   and 527
// (Packed: 8 sequences of 200 rows up to the longest length allowed, log-uniform, x 16 heads, or 32 at 16384.  Their grid has a slot for each tile of
// the longest length, of which about half exist.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "config.h"
#include "dkdv_tile.h"
#include "dq_tile.h"
#include "kernels.h"
#include "smem_limit.h"

namespace s2 {

namespace {

template <int D>
union MergedSmem {
  DkvSmem<D> dkv;
  DqPipeSmem<D> dq;
};

template <int D, bool DENSE, int FINE, bool VARLEN>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 3) void bwd_merged_kernel(const AttnParams p, int keys) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int wg = blockIdx.x;
  if (wg < keys)  // key tiles first: they are the longer ones
    dkdv_tile<D, DENSE, FINE, VARLEN, false>(p, wg, smem_raw);
  else
    dq_tile<D, DENSE, FINE != 0, VARLEN, false>(p, wg - keys, smem_raw);
}

template <int D, bool DENSE, int FINE, bool VARLEN>
hipError_t launch_one(const AttnParams& p, hipStream_t stream) {
  static SmemSet set;  // zero-initialised
  const hipError_t e = set_smem(&bwd_merged_kernel<D, DENSE, FINE, VARLEN>, sizeof(MergedSmem<D>), set);
  if (e != hipSuccess) return e;
  const int keys = (int)p.key_map.grid();  // (a multiple of eight: either part keeps its workgroups' XCDs)
  hipLaunchKernelGGL((bwd_merged_kernel<D, DENSE, FINE, VARLEN>), dim3(keys + p.row_map.grid()), dim3(kThreads), sizeof(MergedSmem<D>), stream, p, keys);
  return hipGetLastError();
}

template <int D>
hipError_t launch_dim(const AttnParams& p, bool dense, hipStream_t stream) {
  if (dense) return launch_one<D, true, 0, false>(p, stream);
  if (p.cu_seqlens) {
    if (p.block_size == 16) return launch_one<D, false, 16, true>(p, stream);
    if (p.block_size == 32) return launch_one<D, false, 32, true>(p, stream);
    return launch_one<D, false, 0, true>(p, stream);
  }
  if (p.block_size == 16) return launch_one<D, false, 16, false>(p, stream);
  if (p.block_size == 32) return launch_one<D, false, 32, false>(p, stream);
  return launch_one<D, false, 0, false>(p, stream);
}

}  // namespace

// The compute units hold 512 (head_dim 128) or 768 (64) of these workgroups at a time.  A launch of a few times as many gains by the start and the
// end that it has once instead of twice; at 4096 that has sunk to what the pass over O and dO on its own costs, and from 8192 on that pass costs
// up to 2 % (measured above; packed batches of up to 8192, whose slots do not all hold a tile, would gain up to 13 % at head_dim 64).
// Two launches also where dK and dV replace K and V (either way round): a key tile writes only what it alone reads, but in one launch the
// dQ tiles read every tile's K and V beside it.
constexpr int kMergedGrid = 4096;
bool bwd_is_merged(const AttnParams& p) {
  const bool in_place = p.dk == p.k || p.dk == p.v || p.dv == p.k || p.dv == p.v;
  return !in_place && p.key_map.grid() + p.row_map.grid() <= kMergedGrid;
}

hipError_t launch_bwd_merged(const AttnParams& p, bool dense, hipStream_t stream) {
  return p.head_dim == 128 ? launch_dim<128>(p, dense, stream) : launch_dim<64>(p, dense, stream);
}

}  // namespace s2
