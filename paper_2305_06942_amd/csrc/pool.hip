// Launch of the pooling kernels (pool_kernels.h).
#include "common.h"

namespace ebag {
namespace {

pool_fn pick(const PoolVariant& k) {
  const bool wide = k.kind == POOL_WIDE;
  switch (k.dtype) {
    case 1: return wide ? pick_pool_wide_f16(k) : pick_pool_f16(k);
    case 2: return wide ? pick_pool_wide_bf16(k) : pick_pool_bf16(k);
    default: return wide ? pick_pool_wide_f32(k) : pick_pool_f32(k);
  }
}

size_t lds_bytes(const PoolVariant& k, int block, int out_floats) {
  return pool_lds_bytes(k.kind != POOL_FAST, k.weighted, block / 64, out_floats);
}

}  // namespace

hipError_t launch_pool(const PoolVariant& k, const PoolArgs& a, int grid, int block, hipStream_t stream) {
  hipLaunchKernelGGL(pick(k), dim3(grid), dim3(block), lds_bytes(k, block, a.out_floats), stream, a);
  return hipGetLastError();
}

int pool_max_wgs_per_cu(const PoolVariant& k, int block, int out_floats) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, pick(k), block, lds_bytes(k, block, out_floats)) != hipSuccess)
    return 0;
  return n;
}

}  // namespace ebag
