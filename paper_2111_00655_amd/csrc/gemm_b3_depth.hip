// 3x3 filters with several depth taps on the split-operand kernels (gemm_b3.h).
#include "gemm_b3.h"

namespace clg {
CLG_B3_INSTANTIATE(9, true, false)
}  // namespace clg
