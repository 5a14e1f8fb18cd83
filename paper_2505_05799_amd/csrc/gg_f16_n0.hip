// Group-GEMM kernel instance: f16 activations, gate|up phase, narrow items.
#include "group_gemm_impl.h"

namespace mxmoe {
MXMOE_GG_LAUNCHER(gg_f16_n0, group_gemm_narrow_kernel, MXMOE_F16, 0)
}  // namespace mxmoe
