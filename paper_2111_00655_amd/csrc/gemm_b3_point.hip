// 1x1 filters and dense layers on the split-operand kernels (gemm_b3.h).
#include "gemm_b3.h"

namespace clg {
CLG_B3_INSTANTIATE(1, false, false)
CLG_B3_INSTANTIATE(1, false, true)
}  // namespace clg
