// dQ launch of the backward that recomputes S and dP (the tile itself: dq_tile.h).
#include <hip/hip_runtime.h>

#include "config.h"
#include "dq_tile.h"
#include "kernels.h"
#include "smem_limit.h"

namespace s2 {

namespace {

template <int D, bool DENSE, bool FINE, bool VARLEN>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 3) void dq_pipe_kernel(const AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  dq_tile<D, DENSE, FINE, VARLEN, true>(p, blockIdx.x, smem_raw);
}

template <int D, bool DENSE, bool FINE, bool VARLEN>
hipError_t launch_one(const AttnParams& p, hipStream_t stream) {
  static SmemSet set;  // zero-initialised
  const hipError_t e = set_smem(&dq_pipe_kernel<D, DENSE, FINE, VARLEN>, sizeof(DqPipeSmem<D>), set);
  if (e != hipSuccess) return e;
  const int grid = (int)p.row_map.grid();
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
