// General pooling kernels for fp32 tables, some of them of rows of more than 32 vectors.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_wide_f32(const PoolVariant& k) { return pick_u<EF32, POOL_WIDE>(k); }

}  // namespace ebag
