// Group-GEMM kernel instance: f16 activations, single linear, narrow items.
#include "group_gemm_impl.h"

namespace mxmoe {
MXMOE_GG_LAUNCHER(gg_f16_nraw, group_gemm_narrow_kernel, MXMOE_F16, kPhaseRaw)
}  // namespace mxmoe
