// Pooling kernels for bf16 tables.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_bf16(const PoolVariant& k) {
  return k.kind == POOL_FAST ? pick_u<EBF16, POOL_FAST>(k) : pick_u<EBF16, POOL_NARROW>(k);
}

}  // namespace ebag
