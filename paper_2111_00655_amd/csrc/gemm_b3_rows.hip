// Transposed convolutions (2x2 taps per phase) and first layers (filter columns folded into
// the channels: 3 or 7 filter rows) on the split-operand kernels (gemm_b3.h).
#include "gemm_b3.h"

namespace clg {
CLG_B3_INSTANTIATE(4, false, false)
CLG_B3_INSTANTIATE(3, true, false)
CLG_B3_INSTANTIATE(8, true, false)
}  // namespace clg
