// Pooling kernels for fp32 tables.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_f32(const PoolVariant& k) {
  return k.kind == POOL_FAST ? pick_u<EF32, POOL_FAST>(k) : pick_u<EF32, POOL_NARROW>(k);
}

}  // namespace ebag
