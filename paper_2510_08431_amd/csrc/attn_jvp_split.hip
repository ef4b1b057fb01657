// Keys in parts: the tile kernels (attn_jvp_mfma.hip with bf16 pairs, attn_jvp_mfma_f32.hip) on calls whose 128-row query
// tiles do not fill the chip's rounds, and the launch that merges what the parts give.
//
// A workgroup takes one query tile against one run of the head's keys and leaves that run's own o, to (fp32), its reference m,
// its sum of weights l (relative to m) and its mu = rowsum(P o tS) in the workspace.  With the weights w_p = l_p e^(m_p) / sum
// of the same, which are the shares of the softmax that fall to the parts,
//     o = sum w_p o_p     mu = sum w_p mu_p     to = sum w_p (to_p + (mu_p - mu) o_p)     lse = log sum l_p e^(m_p)
// exactly (to_p + mu_p o_p is the part's (A + B) / l).
#include "launchers.h"
#include <hip/hip_bf16.h>
#include <algorithm>
#include <cmath>
#include <type_traits>

namespace attn_jvp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int MERGE_THREADS = 256;
constexpr int MAX_PARTS = 8;

// A lane has four columns of a row and all its parts' loads in flight at once (their number is a template parameter): bound by the
// reading of the states.
template <bool BASE2, int PARTS>      // BASE2: m in binades (bf16 kernel), else in nats
__global__ __launch_bounds__(MERGE_THREADS) void merge_parts_kernel(
    const f32x4* __restrict__ o, const f32x4* __restrict__ to, const f32x4* __restrict__ state, void* __restrict__ O, void* __restrict__ tO,
    float* __restrict__ LSE, int Lq, int H, int chunks, long n, int out_bf16, int out_blhd) {
    const long idx = (long)blockIdx.x * MERGE_THREADS + threadIdx.x;
    if (idx >= n) return;
    const long row = idx / chunks;               // (head, query)
    const int chunk = (int)(idx - row * chunks);
    const long bh = row / Lq, q = row - bh * Lq;
    f32x4 st[PARTS], po[PARTS], pt[PARTS];
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
        const long at = (bh * PARTS + p) * Lq + q;
        st[p] = state[at];
        po[p] = o[at * chunks + chunk];
        pt[p] = tO ? to[at * chunks + chunk] : f32x4{};
    }
    // A part whose scores are all -inf has l = 0, and nothing else of it counts.  (l is at least a weight of the reference's
    // size otherwise, or NaN.)
    float m = -INFINITY, l = 0.f, r = 0.f, w[PARTS];
#pragma unroll
    for (int p = 0; p < PARTS; ++p) m = st[p][1] != 0.f ? fmaxf(m, st[p][0]) : m;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
        const float d = st[p][0] - m;
        w[p] = st[p][1] != 0.f ? st[p][1] * (BASE2 ? exp2f(d) : expf(d)) : 0.f;
        l += w[p];
        r = st[p][1] != 0.f ? fmaf(w[p], st[p][2], r) : r;
    }
    const float inv_l = 1.f / l, mu = r * inv_l;
    f32x4 so = {}, st4 = {};
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
        const float f = w[p] * inv_l, dm = st[p][2] - mu;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            so[e] = st[p][1] != 0.f ? fmaf(f, po[p][e], so[e]) : so[e];
            st4[e] = st[p][1] != 0.f ? fmaf(f, fmaf(dm, po[p][e], pt[p][e]), st4[e]) : st4[e];
        }
    }
    if (l == 0.f) {                              // every score -inf: no softmax
        so = f32x4{} * inv_l;
        st4 = so;
    }
    const long out = ((out_blhd ? ((bh / H) * Lq + q) * H + bh % H : row) * chunks + chunk) * 4;
    if (out_bf16) {
        auto store = [&](void* to_, f32x4 x) __attribute__((always_inline)) {
            alignas(8) __hip_bfloat16 b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = __float2bfloat16(x[e]);
            *reinterpret_cast<uint2*>(static_cast<__hip_bfloat16*>(to_) + out) = *reinterpret_cast<const uint2*>(b);
        };
        store(O, so);
        if (tO) store(tO, st4);
    } else {
        *reinterpret_cast<f32x4*>(static_cast<float*>(O) + out) = so;
        if (tO) *reinterpret_cast<f32x4*>(static_cast<float*>(tO) + out) = st4;
    }
    if (chunk == 0) LSE[row] = BASE2 ? (m + log2f(l)) * 0.6931471805599453f : m + logf(l);
}

constexpr size_t up256(size_t n) { return (n + 255) & ~(size_t)255; }

}  // namespace

// How many parts.  Estimated microseconds of a call, from measurements of one chip (69 shapes of 6 to 468 tiles and 17 to 576
// key blocks, parts 1 to 8, all head dimensions; the parts chosen cost 1.7 % more than the best of them on average, and 0.77 of
// the unsplit call):
//   a tile's time is a fixed cost and a time per key block, the latter for a full chip (a quarter less where most of it idles,
//   which leaves the power to the rest); workgroups beyond the compute units wait for the next round;
//   parts add a launch and the states' way to memory and back (4 TB/s in all);
//   the key-split kernel, which the parts replace where it would be slower, has a time per key block and 16 rows.
// Measured, us a call, unsplit -> parts: bf16 d 128, H1 L2000 53 (key-split kernel) -> 33, H4 L1100 54 -> 32, H1 L6000 184 -> 82, H4 L3000
// 113 -> 88; d 64 H1 L6000 129 -> 52; no tangents H2 L3000 57 -> 29; fp32 d 128 H1 L6125 630 -> 189, H8 L700 88 -> 50, H3 L13000 (306
// tiles) 3108 -> 2190; d 64 H4 L2000 119 -> 58.  From about 140 tiles on the bf16 kernels lose (H12 L1560, 156 tiles 73 -> 92).
// Errors against 64 bits do not grow: the sums get shorter (fp32 o 1.0e-6 -> 0.9e-6, 3000 keys), and where the bf16 pairs replace
// the fp16 value path they shrink from 3e-4 to 3e-6.
namespace {

constexpr int UNITS = 256;                            // compute units of the chip the figures are for
constexpr size_t MAX_BYTES = (size_t)160 << 20;       // of states: what the library's own scratch can hold, with room to spare
constexpr double WORTH = 0.92;                        // estimated share of the unsplit time from which on it is not worth it

struct BlockCost {
    double tile, unsplit, keysplit;      // us per key block: a tile in parts; a tile as it runs unsplit from F16_MIN_KEYS on; 16 rows of the key-split kernel
};
BlockCost block_cost(int d, bool f32, bool plain) {
    const int i = d / 32 - 1;
    static const BlockCost bf16_all[4] = {{.95, .58, .28}, {.95, .58, .33}, {1.15, .77, .45}, {1.6, 1.05, .76}};
    static const BlockCost bf16_plain[4] = {{.36, .25, .15}, {.36, .25, .2}, {.47, .33, .22}, {.58, .42, .26}};
    static const BlockCost f32_all[4] = {{1.75, 1.75, .47}, {2.35, 2.35, 1.0}, {3.4, 3.4, 1.27}, {4.4, 4.4, 1.55}};
    static const BlockCost f32_plain[4] = {{.65, .65, .3}, {1.15, 1.15, .5}, {1.3, 1.3, .6}, {1.75, 1.75, .68}};
    return f32 ? (plain ? f32_plain : f32_all)[i] : (plain ? bf16_plain : bf16_all)[i];
}
double rounds_cost(double workgroups, double fixed, double sweep) {
    const double per_unit = workgroups / UNITS, rounds = std::ceil(per_unit);
    return rounds * (fixed + sweep) * (0.75 + 0.25 * per_unit / rounds);
}

size_t bytes_of(long long rows, int d, int parts) {
    return 2 * up256((size_t)rows * parts * d * 4) + up256((size_t)rows * parts * 16);
}

}  // namespace

KeySplit plan_split(int B, int H, int Lq, int Lkv, int d, bool f32, bool tangents, bool key_tangents) {
    KeySplit best;
    const int q_tiles = (Lq - 1) / MFMA_TILE_ROWS + 1;
    if ((d != 32 && d != 64 && d != 96 && d != 128) || (double)q_tiles * B * H > 4 * UNITS) return best;
    const long long rows = (long long)B * H * Lq, tiles = (long long)q_tiles * B * H;
    const int blocks = (Lkv - 1) / 32 + 1;
    const BlockCost c = block_cost(d, f32, !tangents);
    const double fixed = f32 ? 12 : 10;
    const long long groups = (long long)((Lq - 1) / 16 + 1) * B * H;
    double unsplit;
    if (groups <= (long long)keysplit_groups_per_unit(d, f32, tangents, key_tangents) * UNITS)
        unsplit = 8 + c.keysplit * blocks * std::max(1.0, (double)groups / UNITS);
    else if (!f32 && Lkv >= F16_MIN_KEYS)      // the fp16 value path: its pre-pass, and more to do at a tile's start and end
        unsplit = 34 + rounds_cost((double)tiles, 5, blocks * c.unsplit);
    else
        unsplit = rounds_cost((double)tiles, fixed, blocks * c.tile);
    double least = WORTH * unsplit;
    for (int parts = 2; parts <= MAX_PARTS; ++parts) {
        const int run = (blocks + parts - 1) / parts;      // key blocks of a part
        if (run < 4 || (blocks + run - 1) / run != parts || bytes_of(rows, d, parts) > MAX_BYTES) continue;
        const double cost = rounds_cost((double)tiles * parts, fixed, run * c.tile) + 7 + (double)rows * parts * d * (tangents ? 8 : 4) / 4e6;
        if (cost < least) {
            least = cost;
            best = KeySplit{parts, run};
        }
    }
    return best;
}

size_t split_bytes(int B, int H, int Lq, int Lkv, int d, bool f32) {
    size_t most = 0;          // (whichever tangents the call has)
    for (int tangents = 0; tangents < 3; ++tangents) {
        const KeySplit split = plan_split(B, H, Lq, Lkv, d, f32, tangents > 0, tangents > 1);
        const size_t n = split.parts > 1 ? bytes_of((long long)B * H * Lq, d, split.parts) : 0;
        most = n > most ? n : most;
    }
    return most;
}

PartStates part_states(const Problem& p) {
    if (p.split.parts <= 1) return PartStates{p.o, p.to, nullptr, p.out_dtype, p.out_layout};
    const size_t rows = (size_t)p.B * p.H * p.Lq * p.split.parts, values = up256(rows * p.d_out * 4);
    char* at = static_cast<char*>(p.workspace);
    return PartStates{at, at + values, reinterpret_cast<float*>(at + 2 * values), 0, 0};
}

hipError_t launch_merge_parts(const Problem& p, const PartStates& ps) {
    const int chunks = p.d_out / 4;
    const long n = (long)p.B * p.H * p.Lq * chunks;
    const long grid = (n + MERGE_THREADS - 1) / MERGE_THREADS;
    auto launch = [&](auto parts) {
        constexpr int PARTS = decltype(parts)::value;
        const bool bf16 = p.in_dtype == 0;
        hipLaunchKernelGGL(bf16 ? (merge_parts_kernel<true, PARTS>) : (merge_parts_kernel<false, PARTS>), dim3((unsigned)grid), dim3(MERGE_THREADS), 0,
                           p.stream, (const f32x4*)ps.o, (const f32x4*)ps.to, (const f32x4*)ps.state, p.o, p.tq ? p.to : nullptr, p.lse, p.Lq, p.H,
                           chunks, n, bf16 ? p.out_dtype : 0, p.out_layout);
    };
    static_assert(MAX_PARTS == 8, "one case each");
    switch (p.split.parts) {
        case 2: launch(std::integral_constant<int, 2>{}); break;
        case 3: launch(std::integral_constant<int, 3>{}); break;
        case 4: launch(std::integral_constant<int, 4>{}); break;
        case 5: launch(std::integral_constant<int, 5>{}); break;
        case 6: launch(std::integral_constant<int, 6>{}); break;
        case 7: launch(std::integral_constant<int, 7>{}); break;
        case 8: launch(std::integral_constant<int, 8>{}); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace attn_jvp
