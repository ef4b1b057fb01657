// The bf16 matrix-core kernel at head dimension 64 (sources of their own, so that the instantiations compile side by side; 32 runs on copies padded to 64 columns).
#include "mfma_kernel.h"

namespace attn_jvp {

hipError_t launch_mfma_bf16_64(const Problem& p) { return launch_dh<64>(p); }

}  // namespace attn_jvp
