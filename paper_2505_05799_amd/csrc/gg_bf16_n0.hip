// Group-GEMM kernel instance: bf16 activations, gate|up phase, narrow items.
#include "group_gemm_impl.h"

namespace mxmoe {
MXMOE_GG_LAUNCHER(gg_bf16_n0, group_gemm_narrow_kernel, MXMOE_BF16, 0)
}  // namespace mxmoe
