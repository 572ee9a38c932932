// gemm_direct.hip -- the few-output BFP GEMM (kernel in gemm_direct.h) for
// groups of 16, every operand format.
#include "gemm_direct.h"

namespace fastbfp {

FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 1, 1, 16)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 1, 2, 16)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 2, 1, 16)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 2, 2, 16)

}  // namespace fastbfp
