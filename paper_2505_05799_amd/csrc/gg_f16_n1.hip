// Group-GEMM kernel instance: f16 activations, down phase, narrow items.
#include "group_gemm_impl.h"

namespace mxmoe {
MXMOE_GG_LAUNCHER(gg_f16_n1, group_gemm_narrow_kernel, MXMOE_F16, 1)
}  // namespace mxmoe
