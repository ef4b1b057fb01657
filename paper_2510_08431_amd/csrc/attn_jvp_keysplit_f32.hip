// The key-split kernel on fp32 inputs.
#include "keysplit_kernel.h"

namespace attn_jvp {

hipError_t launch_keysplit_f32(const Problem& p) { return launch_dim<float>(p); }

}  // namespace attn_jvp
