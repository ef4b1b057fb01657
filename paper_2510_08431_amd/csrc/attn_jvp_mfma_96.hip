// The bf16 matrix-core kernel at head dimension 96 (sources of their own, so that the instantiations compile side by side).
#include "mfma_kernel.h"

namespace attn_jvp {

hipError_t launch_mfma_bf16_96(const Problem& p) { return launch_dh<96>(p); }

}  // namespace attn_jvp
