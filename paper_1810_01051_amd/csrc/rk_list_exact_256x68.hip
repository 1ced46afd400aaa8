// Exact family (d = 256, q = 2^61 - 1; hash dump), single-bucket kernels of one
// key and of two, tile geometry 256x68 (workgroup size x windows per thread): one
// geometry per translation unit, so that the exact kernels compile in parallel.
#include "rk_scan.h"

namespace rk {
RK_INSTANTIATE_LIST(kFamExact, 0)
RK_INSTANTIATE_LIST(kFamExactFew, 0)
}  // namespace rk
