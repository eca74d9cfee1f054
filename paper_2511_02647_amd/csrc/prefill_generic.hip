// General prefill attention kernel (plain ALU, fp32 arithmetic): one wavefront per
// (query row, query head).  It reads token-granular keep flags as they are and needs no
// workspace, so it takes the keep-list calls that come without one (fp32, and bf16 with head
// dimensions other than 64 and 128); everything else runs on the matrix cores.
#include "common.h"
#include "row_walk.h"

namespace fedattn {

namespace {

template <typename T>
__global__ __launch_bounds__(256) void prefill_rows_kernel(PrefillArgs a) {
  __shared__ float q_s[4][256];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t pair = (int64_t)blockIdx.x * 4 + wave;
  const int64_t n_pairs = (int64_t)a.total * a.Hq;
  if (pair >= n_pairs) return;  // only wave-level synchronisation below
  const int block = blockIdx.y;
  const int i = (int)(pair / a.Hq);
  const int h = (int)(pair % a.Hq);
  const bool is_sync = a.sync_override >= 0 ? (a.sync_override != 0)
                                            : sync_block_rule(a.sync_interval, a.block_idx0 + block);
  const T* q = reinterpret_cast<const T*>(a.q) + (int64_t)block * a.q_block_stride;
  float* qs = q_s[wave];
  for (int d = lane; d < a.D; d += 64) qs[d] = RowLoad<T>::at(q + ((int64_t)i * a.Hq + h) * a.D + d);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  prefill_row<T, false>(a, block, is_sync, i, h, [&](int d) { return qs[d]; }, [](int) { return true; });
}

}  // namespace

hipError_t launch_prefill_generic(const PrefillArgs& a, int n_blocks, int dtype, hipStream_t s) {
  const int64_t n_pairs = (int64_t)a.total * a.Hq;
  if (n_pairs == 0 || n_blocks == 0) return hipSuccess;
  dim3 grid((unsigned)((n_pairs + 3) / 4), (unsigned)n_blocks, 1);
  if (dtype == FEDATTN_F32)
    hipLaunchKernelGGL(prefill_rows_kernel<float>, grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(prefill_rows_kernel<uint16_t>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace fedattn
