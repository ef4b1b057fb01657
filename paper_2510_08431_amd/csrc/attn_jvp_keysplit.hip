// The key-split kernel (keysplit_kernel.h) on bf16 inputs, and the rule that takes calls to it.
#include "keysplit_kernel.h"

namespace attn_jvp {

// Where this kernel beats the tile kernels, in workgroups (16 query rows each) per compute unit.  Both times grow alike with the
// keys from 32 to 2048 (8 heads, whole calls, tile kernel over this one, at the workgroups per unit named):
//   d = 32    bf16 4: 1.18 to 2.3, fp32 3: 0.99 (32 keys) to 1.5, 4: 0.93 to 1.2
//   two workgroups share a unit (bf16 up to 128, fp32 up to 64), 2: 1.05 to 1.5, 3: 0.73 to 1.4; bf16 d = 128 with all tangents 1:
//             1.33 to 1.52, 2: 0.93 to 1.18
//   one does (fp32 96, 128), 1: 1.6 to 2.2, 2: 0.91 to 1.13 with tangents, 1.2 to 1.44 without
// and at most 64 workgroups 1.23 to 3.5.  (Tile kernels on all keys; where a workspace is there, plan_split compares it with tiles on
// keys in parts.)
int keysplit_groups_per_unit(int d, bool f32, bool tangents, bool key_tangents) {
    return d == 32 ? (f32 ? 3 : 4) : f32 ? (d == 64 || !tangents ? 2 : 1) : d == 128 && key_tangents ? 1 : 2;
}
hipError_t keysplit_preferred(const Problem& p, bool* yes) {
    int dev = 0, cus = 0;
    const hipError_t e = device_cus(&dev, &cus);
    if (e != hipSuccess) return e;
    const long long workgroups = (long long)((p.Lq + BR - 1) / BR) * p.B * p.H;
    *yes = workgroups <= (long long)keysplit_groups_per_unit(p.d, p.in_dtype == 1, p.tq != nullptr, p.tk != nullptr) * cus;
    return hipSuccess;
}

hipError_t launch_keysplit(const Problem& p) {
    return p.in_dtype == 1 ? launch_keysplit_f32(p) : launch_dim<__hip_bfloat16>(p);
}

}  // namespace attn_jvp
