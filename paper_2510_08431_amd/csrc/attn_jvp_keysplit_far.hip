// The key-split kernel on bf16 inputs whose rows are far apart ([B,L,H,d] with 2^25 / d heads or more).
#include "keysplit_kernel.h"

namespace attn_jvp {
namespace {

template <int D>
hipError_t launch_far(const Problem& p) {
    using T = __hip_bfloat16;
    return !p.tq ? launch_waves<T, D, TAN_NONE, 4, 2, true>(p) : !p.tk ? launch_waves<T, D, TAN_QUERY, 4, 2, true>(p) : launch_waves<T, D, TAN_ALL, 4, 2, true>(p);
}

}  // namespace

hipError_t launch_keysplit_far(const Problem& p) {
    switch (p.d) {
        case 32: return launch_far<32>(p);
        case 64: return launch_far<64>(p);
        case 96: return launch_far<96>(p);
        case 128: return launch_far<128>(p);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace attn_jvp
