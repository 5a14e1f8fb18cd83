// Group-GEMM kernel instance: bf16 activations, single linear, narrow items.
#include "group_gemm_impl.h"

namespace mxmoe {
MXMOE_GG_LAUNCHER(gg_bf16_nraw, group_gemm_narrow_kernel, MXMOE_BF16, kPhaseRaw)
}  // namespace mxmoe
