// Pooling kernels for bf16 tables.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_bf16(const PoolVariant& k) { return pick_u<EBF16>(k); }

}  // namespace ebag
