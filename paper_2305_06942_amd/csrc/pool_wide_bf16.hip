// General pooling kernels for bf16 tables, some of them of rows of more than 32 vectors.
#include "pool_kernels.h"

namespace ebag {

pool_fn pick_pool_wide_bf16(const PoolVariant& k) { return pick_u<EBF16, POOL_WIDE>(k); }

}  // namespace ebag
