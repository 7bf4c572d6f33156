// Pooling kernels for fp32 tables.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_f32(const PoolVariant& k) { return pick_u<EF32>(k); }

}  // namespace ebag
