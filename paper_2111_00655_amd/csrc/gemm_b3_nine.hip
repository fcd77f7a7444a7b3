// 3x3 filters on the split-operand kernels (gemm_b3.h).
#include "gemm_b3.h"

namespace clg {
CLG_B3_INSTANTIATE(9, false, false)
}  // namespace clg
