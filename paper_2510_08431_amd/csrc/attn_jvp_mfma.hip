// The bf16 matrix-core kernel (mfma_kernel.h) at head dimension 128, and which calls and which tier it takes.
#include "mfma_kernel.h"

namespace attn_jvp {

// scale > 0: the kernel masks padded keys with a raw score of -inf and takes row maxima before scaling.
// tk and tv are either both given or both absent (zero key/value tangents); single bf16 weights (FAST) are not built
// for the latter.
// Head dimensions 128, 96 and 64 are built natively; 32 runs on zero-padded copies (64 columns), which need the caller's
// workspace.  96 is taken with such a workspace only, too: without one the interface refuses it.
static bool workspace_head_dim(const Problem& p) {
    return (p.d == 32 || p.d == 96) && p.workspace != nullptr &&
           (reinterpret_cast<uintptr_t>(p.workspace) & 255u) == 0 &&
           p.workspace_bytes >= pad_workspace_bytes(p.B, p.H, p.Lq, p.Lkv, p.d);
}
bool mfma_bf16_supports(const Problem& p) {
    const bool zt = p.tk == nullptr && p.tv == nullptr;     // (the API admits absent tangents only as tk+tv or tq+tk+tv)
    return p.in_dtype == 0 && (p.d == 128 || p.d == 64 || workspace_head_dim(p)) && p.scale > 0.f && !(zt && (p.flags & 1));
}

// fp16 value path when the caller lent enough scratch (and did not ask for another variant) and the call is
// large enough to amortise its per-call pre-pass (see F16_MIN_KEYS)
bool mfma_f16_path(const Problem& p, int cus) {
    const long long tiles = (long long)((p.Lq + BR - 1) / BR) * p.B * p.H;
    return !(p.flags & 3) && p.split.parts == 1 && p.workspace != nullptr && (long long)p.B * p.H <= 65535 &&   // pre-pass grid.y
           (p.Lkv >= F16_MIN_KEYS || (p.flags & 4) ||
            (p.Lkv >= F16_MIN_KEYS_MANY_TILES && tiles >= (long long)F16_MANY_TILES_PER_CU * cus)) &&
           p.workspace_bytes >= f16_workspace_bytes(p.B, p.H, p.Lq, p.Lkv, p.d) &&
           (reinterpret_cast<uintptr_t>(p.workspace) & 255u) == 0;
}

hipError_t mfma_bf16_takes_f16(const Problem& p, bool* yes) {
    int dev = 0, cus = 0;
    const hipError_t e = device_cus(&dev, &cus);
    if (e != hipSuccess) return e;
    Problem padded = p;
    if (p.d == 32) {      // (what launch_pad_inputs leaves; supported only with room for the copies)
        padded.d = padded_head_dim_of(p.d);
        const size_t copies = pad_workspace_bytes(p.B, p.H, p.Lq, p.Lkv, p.d);
        padded.workspace = static_cast<char*>(p.workspace) + copies;
        padded.workspace_bytes = p.workspace_bytes - copies;
    }
    *yes = mfma_f16_path(padded, cus);
    return hipSuccess;
}

hipError_t launch_mfma_bf16(const Problem& p) {
    if (!mfma_bf16_supports(p)) return hipErrorInvalidValue;
    return p.d <= 64 ? launch_mfma_bf16_64(p) : p.d == 96 ? launch_mfma_bf16_96(p) : launch_dh<128>(p);     // 32 runs on copies padded to 64 columns
}

}  // namespace attn_jvp
