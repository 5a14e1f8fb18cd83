// Group-GEMM kernel instance: bf16 activations, down phase, narrow items.
#include "group_gemm_impl.h"

namespace mxmoe {
MXMOE_GG_LAUNCHER(gg_bf16_n1, group_gemm_narrow_kernel, MXMOE_BF16, 1)
}  // namespace mxmoe
