// Pooling kernels for fp16 tables.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_f16(const PoolVariant& k) { return pick_u<EF16>(k); }

}  // namespace ebag
