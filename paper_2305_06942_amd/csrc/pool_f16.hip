// Pooling kernels for fp16 tables.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_f16(const PoolVariant& k) {
  return k.kind == POOL_FAST ? pick_u<EF16, POOL_FAST>(k) : pick_u<EF16, POOL_NARROW>(k);
}

}  // namespace ebag
