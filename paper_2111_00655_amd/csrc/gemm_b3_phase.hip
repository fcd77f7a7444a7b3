// Transposed convolutions with 2x2 taps per phase on the split-operand kernels (gemm_b3.h).
#include "gemm_b3.h"

namespace clg {
CLG_B3_INSTANTIATE(4, false, false)
}  // namespace clg
