// gemm_direct_g32.hip -- the few-output BFP GEMM (kernel in gemm_direct.h) for
// groups of 32, every operand format.
#include "gemm_direct.h"

namespace fastbfp {

FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 1, 1, 32)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 1, 2, 32)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 2, 1, 32)
FASTBFP_DIRECT_ALL(FASTBFP_DIRECT_INSTANTIATE, 2, 2, 32)

}  // namespace fastbfp
