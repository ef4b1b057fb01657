// The key-split kernel at head dimension 256 (sources of their own, so that the instantiations compile side by side).
#include "keysplit_kernel.h"

namespace attn_jvp {

hipError_t launch_keysplit_256(const Problem& p) { return p.in_dtype == 1 ? launch_tan<float, 256>(p) : launch_tan<__hip_bfloat16, 256>(p); }

}  // namespace attn_jvp
