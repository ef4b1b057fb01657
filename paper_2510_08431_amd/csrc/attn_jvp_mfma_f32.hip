// Matrix-core streaming kernel for attention forward + JVP (paper App. C.1, Alg. 2) on fp32 inputs, gfx950; head dims
// 32, 64, 96, 128.
//
// The fp32 MFMAs run at a sixteenth of the rate of the 16-bit ones and share the vector ALU's arithmetic, so every
// product is formed from operands SPLIT into two fp16 terms instead: x = 2^e (hi + lo) with hi = fp16(x 2^-e), lo =
// fp16(x 2^-e - hi), and a b = hi hi + hi lo + lo hi, three 16-bit MFMAs with fp32 accumulation.  hi + lo carries 22 to
// 23 bits, the dropped lo lo term is below 2^-22 of the product: rounding of the same size as that of the fp32 score
// sums, and three (not sixteen) rounded additions per accumulator and 16 keys make the accumulators' own error smaller
// than that of fp32 MFMAs, which take one per two keys.
// Powers of two keep everything inside the fp16 range (they add no rounding):
//   Q, tQ rows and K, tK rows: each row by its own largest element, to [2^12, 2^13).  The factors are undone on the
//     scores, per lane for the query and per register for the key.
//   V, tV: by the head's first key block, its largest |V| to [2^11, 2^12); tV shares V's factor times 2^eH.
//   weights: P~ 2^12 with P~ = exp(S - m) against a row reference m that trails the row maximum by at most 2.68 nats
//     (so that keys 25 nats below the maximum still count); H~ 2^(12 - eH) with 2^eH from the first block's tangent
//     scores and |tV| / |V|.
// Values that these scales do not suit send the workgroup's tile to a pass with fp32 MFMAs (fp32_tile), as do infinities
// and NaN in the inputs.  Too large a value becomes inf in fp16 and shows in l, r or the accumulators.  Too small ones would
// sink into fp16 subnormals unseen: the conversion looks at the largest of each eight values of V and tV that it splits, and
// a row whose results come out small against what the split resolves is found at the end (the weights of keys that hold the
// scale up may be nil).  Likewise the rows of Q, tQ, K and tK are looked at for elements far below their row's largest; where
// it is keys, their weights decide.  What the conversion sees ends the sweep soon, what the end of the sweep sees
// costs the sweep on top (B2 H16 L4096 d128: 6.4 ms for fp32 products alone).  l and r are summed in fp32 from the
// unrounded weights.
//
// Work split: a workgroup of 4 waves owns 128 query rows, 32 per wave; key blocks of BC = 32 rows.  Products are taken
// transposed, S^T = K Q^T and O^T += V^T P~^T, on v_mfma_f32_32x32x16_f16: the query index is the MFMA column (lane %
// 32), each lane holds 16 of the 32 scores of ONE query row, and the split weights are the B operands of the value
// products as they stand.
//
// The split planes of K, tK (row-major) and V, tV (transposed [D][32 keys], keys in the order the score MFMAs leave
// them in a lane's registers) go through two LDS stages each.  The four waves fetch fp32 blocks two (K) and one (V)
// blocks ahead into registers and convert them behind the score MFMAs; behind the value MFMAs run the softmax and
// weight splitting of the NEXT block.  One barrier per block.  Bound by the matrix pipe at D = 128 (144 MFMAs per wave
// and block, about 590 other vector instructions, 40 of them the checks of the scales, which cost 1 to 3 % here, 6 on
// few blocks): B2 H16 L4096 d128 2.19 ms = 376 TFLOP/s counted (6.40 ms with fp32 MFMAs), the matrix pipe busy 56 % of
// the time; d = 64 1.20 ms (3.14), d = 32 0.85 (1.65).  Errors against 64 bits are 0.6 to 0.7 of those of the fp32-MFMA kernel in o and to, the same in lse.
#include "launchers.h"
#include <type_traits>
#include <utility>
#include <stdint.h>

namespace attn_jvp {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int BR = 128;          // query rows per workgroup
constexpr int BC = 32;           // key rows per block
constexpr int NTHREADS = 256;
constexpr int TAN_NONE = 0;      // no tangents: O, lse only
constexpr int TAN_QUERY = 1;     // tQ only (tK = tV = 0)
constexpr int TAN_ALL = 2;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr int ROW_TOP = 12;      // rows of Q, tQ, K, tK: largest element in [2^12, 2^13)
constexpr int EVEN_SPAN = 15;    // a row's eight neighbouring elements are known to 2^-22 of their largest if that is 2^-15 of the
                                 // row's or more (2^-3 scaled); a row with smaller ones is called uneven
constexpr float UNEVEN_SHARE = 0x1p-32f;    // share of a row's weights that uneven keys may have (2^-20 e^-8)
constexpr int V_TOP = 11;        // first block of V: largest element in [2^11, 2^12), 4 binades in hand for later blocks
constexpr int V_FLOOR = -3;      // eight keys of a column are known to 2^-22 of their largest if that is 2^-3 or more, scaled
constexpr uint32_t V_AMPLE = 5u << 23;    // 2^2 in units of that: where V is as large tV may be smaller, beside H~ V its share of tO is known well enough
constexpr int V_HITS = 4;        // blocks in which a column has to be found below: one value beside seven zeros is small now and then
constexpr float ONE_KEY = 1.5f;           // sum of a row's weights over the largest of them, below which the row is one key's,
constexpr float ONE_KEY_GAIN = 256.f;     // ... and what its A + B may then be smaller by
constexpr float ROW_FLOOR = 16384.f;      // (2^7)^2: see the check at the end of the sweep
constexpr int T_HEADROOM = 4;    // the first block's largest tangent score is scaled to [2^-4, 2^-3)
constexpr float P_GAIN = 4096.f;          // the split weights are P~ 2^12 ...
constexpr float P_SLACK = 2.68f;          // ... and stay below 2^16: nats by which a block may exceed the reference before it moves
constexpr float FP32_SLACK = 32.f;        // fp32_tile: nats by which scores may exceed the reference

#define FENCE() __builtin_amdgcn_sched_barrier(0)      // no instruction is scheduled across this point

// Score products with the result in ARITHMETIC registers (the vector ALU reads every score; left to itself the compiler
// puts the results of MFMAs into accumulation registers, which Q, tQ and the accumulators fill, and spills).  It does
// not see inside: SCORE_RESULTS_LAND supplies the 12 wait states an 8-pass MFMA needs before its result may be read,
// and the statements that follow it keep every result register live until then.  The build checks the compiled
// assembly for both (lint_mfma_asm.py).  SMFMA0 starts a chain (C = 0), SMFMA continues it.
#define SMFMA0(a, b, c) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "a"(b))
#define SMFMA(a, b, c) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "a"(b))
#define SCORE_RESULTS_LAND() asm volatile("s_nop 7\n\ts_nop 3" ::: "memory")

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {      // f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
    static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ float xhalf_max(float x) {   // max of lane l and lane l^32, in both
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ f32x16 mfma16(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t pack_f16(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}
// Splitting a pair: hi = fp16(x s) of both halves, lo = fp16(x s - hi), with s a power of two, so that x s and the
// difference (one mixed-precision fused multiply-add) are exact.  (v_fma_mixlo_f16 / mixhi_f16 would round to a half
// register directly, in fewer instructions, but take 12 and 9 cycles each, the packed conversion 8 for both halves.)
__device__ __forceinline__ uint32_t split_hi(float x0, float x1, float s) { return pack_f16(x0 * s, x1 * s); }
__device__ __forceinline__ uint32_t split_lo(float x0, float x1, float s, uint32_t h) {
    float r0, r1;
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,0] op_sel_hi:[0,0,1]" : "=v"(r0) : "v"(x0), "v"(s), "v"(h));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(r1) : "v"(x1), "v"(s), "v"(h));
    return pack_f16(r0, r1);
}
// max(|a|, |b|, |c|) (as assembly: fmaxf would first canonicalise every operand that comes from memory); a NaN is passed over
__device__ __forceinline__ float max_abs3(float a, float b, float c) {
    float d;
    asm volatile("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ float max3(float a, float b, float c) {
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
template <int CTRL>
__device__ __forceinline__ float max_dpp(float x) {      // x >= 0 on every lane
    const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true);
    return __int_as_float(max(__float_as_int(x), y));    // non-negative floats order as integers
}
// biased exponent of a largest element, kept where 2^(ROW_TOP - e), 2^(e - ROW_TOP) and their like are normal numbers
__device__ __forceinline__ int top_exponent(float mx) {
    const int e = __float_as_int(mx) >> 23;
    return e < 24 ? 24 : e;
}
__device__ __forceinline__ float pow2(int biased) { return __int_as_float(biased << 23); }
// is the largest of some elements of a row, not zero, below what the row's scale suits?  (factor: pow2(its exponent - ROW_TOP))
__device__ __forceinline__ bool below_span(float own, float factor) {
    return __float_as_uint(own) - 1 < __float_as_uint(factor) - ((uint32_t)(EVEN_SPAN - ROW_TOP) << 23) - 1;      // (a zero wraps around)
}
__device__ __forceinline__ u32x4 lds_read_b128(uint32_t addr) {
    return *reinterpret_cast<__attribute__((address_space(3))) const u32x4*>((uintptr_t)addr);
}
__device__ __forceinline__ void lds_write_b128(uint32_t addr, u32x4 v) {
    *reinterpret_cast<__attribute__((address_space(3))) u32x4*>((uintptr_t)addr) = v;
}
__device__ __forceinline__ float lds_read_f32(uint32_t addr) {
    return *reinterpret_cast<__attribute__((address_space(3))) const float*>((uintptr_t)addr);
}
__device__ __forceinline__ void lds_write_f32(uint32_t addr, float v) {
    *reinterpret_cast<__attribute__((address_space(3))) float*>((uintptr_t)addr) = v;
}
__device__ __forceinline__ f32x4 lds_read_f32x4(uint32_t addr) {
    return *reinterpret_cast<__attribute__((address_space(3))) const f32x4*>((uintptr_t)addr);
}
__device__ __forceinline__ f32x2 lds_read_f32x2(uint32_t addr) {
    return *reinterpret_cast<__attribute__((address_space(3))) const f32x2*>((uintptr_t)addr);
}

template <int D, int TAN>
struct Geo {
    static constexpr int PLANE = BC * D * 2;                    // one fp16 plane of a tensor's block
    static constexpr int PLANES = TAN == TAN_ALL ? 4 : 2;       // X hi, X lo (, tX hi, tX lo)
    static constexpr int STAGE = PLANES * PLANE;                // K side or V side
    static constexpr int V_BASE = 2 * STAGE;                    // two stages of K, then two of V
    static constexpr int F_BASE = 4 * STAGE;                    // row factors: [2 stages][K, tK][32] floats
    static constexpr int RED_BASE = F_BASE + 2 * 2 * BC * 4;    // scratch of the workgroup's reductions and votes
    static constexpr int NOTE_BASE = RED_BASE + 64;             // [block % 4]: bits of its uneven keys; not 0: the sweep is to end
    static constexpr int DUMMY_BASE = NOTE_BASE + 32;
    static constexpr int LDS_BYTES = DUMMY_BASE + 256 + 2 * 2 * BC * 4;
    static constexpr int WG_PER_CU = TAN == TAN_NONE || (TAN == TAN_QUERY && D == 32) ? 2 : 1;     // as the registers allow
    // The last block's value products alone, or as one more iteration with the scores and conversions of a block past the end, which takes
    // twice the time: alone where that pays.  At head dimensions 32 and 64 with all tangents or none it made the loop itself 1 to 4 %
    // slower (H24 L3000 d32 478 -> 501 us a call, without tangents H8 L2668 d64 97.5 -> 100.5).
    static constexpr bool LAST_ALONE = D >= 96 || TAN == TAN_QUERY;
    static constexpr int LPR = D == 96 ? 16 : D / 8;            // lanes that convert one K row, 8 elements each (D = 96: 12 of 16)
    static constexpr int K_ROWS = NTHREADS / LPR < BC ? NTHREADS / LPR : BC;    // rows per conversion pass
    static constexpr int K_PASSES = BC / K_ROWS;
    static constexpr int V_PASSES = (D + 63) / 64;              // a V pass: 64 columns (lanes) x 4 groups of 8 keys (waves)
    // chunk swizzle of a K row (16-byte chunks): the 16 lanes a 128-bit read serves together cover all banks
    static __device__ __forceinline__ int k_swizzle(int row) {
        return D == 128 ? (row & 15) : D == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3);
    }
};

// 128-bit direct-to-LDS load: 64 lanes x 16 B land at lds_base + 16 * lane (M0 carries lds_base); uniform 64-bit base
// in scalar registers plus a per-lane 32-bit byte offset.  Inline assembly so that the pass below keeps its own account of
// these loads: an explicit wait plus the barrier at the end of each block publish a stage before anyone reads it.
__device__ __forceinline__ void load_lds_b128(const void* uniform_base, uint32_t lane_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(lane_off), "s"(uniform_base) : "memory");
}

// Alg. 2 in fp32 throughout for the workgroup's 128 query rows, v_mfma_f32_32x32x2_f32: what the split products cannot do.
//   score step 4u + e (u < D/8, e < 4): A = K[key = c][8u + 4g + e], B = Q[query = c][8u + 4g + e]
//   value step t < 16, column block n: A = V[key = 8(t/4) + 4g + t%4][32n + c], B = weight register t
// Blocks of 32 keys go through two LDS stages as fp32, by direct-to-LDS loads; chunk x of a row sits at x ^ (row & 7), which
// spreads the reads of either side over the banks.  Operands are read one step ahead; the weights of step t + 1 are computed
// behind step t's products.  The row reference trails the running maximum by up to FP32_SLACK nats.  On entry the workgroup
// has passed a barrier behind its last use of the LDS; l and r come back as this lane's part of the row sums.
// (B2 H16 L4096 d128: 6.4 ms if every tile comes here; with unstaged loads it took 12.5.)
template <int D, int TAN>
__device__ __forceinline__ void fp32_tile(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ tQ, const float* __restrict__ tK, const float* __restrict__ tV,
    long q_row, long kv_base, long row_elems, int Lkv, float scale, uint32_t lds0, int lane, int wave,
    f32x16 (&acc_o)[D / 32], f32x16 (&acc_t)[TAN != TAN_NONE ? D / 32 : 1], float& m, float& l, float& r) {
#pragma clang fp contract(off)
    constexpr bool TANGENT = TAN != TAN_NONE, KV_TANGENT = TAN == TAN_ALL;
    constexpr int CH = D / 4;                        // 16-byte chunks per row
    constexpr int TILE = BC * D * 4;                 // bytes of a tensor's staged block
    constexpr int PT = BC * CH / NTHREADS;           // chunks each lane moves per tensor and block
    constexpr int NT = KV_TANGENT ? 4 : 2;           // tensors staged: K, V (, tK, tV)
    constexpr int NC = D / 32;
    constexpr int T_K = 0, T_V = 1, T_TK = 2, T_TV = 3;
    static_assert(2 * PT < D / 8 && 2 * PT < 16, "a block's parts fit the steps they are issued behind");
    const int c = lane & 31, g = lane >> 5;

    f32x4 q[D / 8], tq[TANGENT ? D / 8 : 1];         // columns 8u + 4g .. + 3 of the lane's row
#pragma unroll
    for (int u = 0; u < D / 8; ++u) {
        q[u] = *reinterpret_cast<const f32x4*>(Q + q_row + 4 * g + 8 * u);
        if constexpr (TANGENT) tq[u] = *reinterpret_cast<const f32x4*>(tQ + q_row + 4 * g + 8 * u);
    }
#pragma unroll
    for (int u = 0; u < D / 8; ++u) asm volatile("" : "+a"(q[u]));       // only MFMAs read it

    uint32_t g_off[PT];                              // byte offsets of the lane's chunks from the block's first row
    int s_row[PT];
    const int tid = 64 * wave + lane;
#pragma unroll
    for (int n = 0; n < PT; ++n) {
        const int idx = tid + NTHREADS * n, row = idx / CH, pc = idx % CH;
        s_row[n] = row;
        g_off[n] = (uint32_t)((row * row_elems + 4 * (pc ^ (row & 7))) * (long)sizeof(float));
    }
    auto stage_part = [&](const float* base, int j0, int stage, int tensor, int n) __attribute__((always_inline)) {
        const char* blk = reinterpret_cast<const char*>(base + kv_base + (long)j0 * row_elems);
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)((stage * NT + tensor) * TILE + (64 * wave + NTHREADS * n) * 16));
        // rows past the end re-read the block's first row (their weight is zero)
        const bool dead = j0 + BC > Lkv && j0 + s_row[n] >= Lkv;
        load_lds_b128(blk, dead ? g_off[n] - (uint32_t)(s_row[n] * row_elems * (long)sizeof(float)) : g_off[n], dst);
    };
    auto stage_in = [&](const float* base, int j0, int stage, int tensor) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < PT; ++n) stage_part(base, j0, stage, tensor, n);
    };
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        acc_o[n] = f32x16{};
        if constexpr (TANGENT) acc_t[n] = f32x16{};
    }
    m = -INFINITY; l = 0.f; r = 0.f;
    const int n_blocks = (Lkv + BC - 1) / BC;
    stage_in(K, 0, 0, T_K);
    stage_in(V, 0, 0, T_V);
    if constexpr (KV_TANGENT) {
        stage_in(tK, 0, 0, T_TK);
        stage_in(tV, 0, 0, T_TV);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll 1
    for (int blk = 0; blk < n_blocks; ++blk) {
        const int cur = blk & 1, nxt = cur ^ 1, j0 = blk * BC;
        const bool has_next = blk + 1 < n_blocks;
        // ---- S^T = K Q^T, tS^T = K tQ^T + tK Q^T (three chains in turn); the next block's K, tK travel meanwhile
        f32x16 s = f32x16{}, ts = f32x16{}, ts2 = f32x16{};
        {
            uint32_t lk[4];                          // chunk (2u + g) ^ (c & 7) = 8 (u/4) + ((2 (u%4) + g) ^ (c & 7))
#pragma unroll
            for (int w = 0; w < 4; ++w) lk[w] = lds0 + (uint32_t)((cur * NT + T_K) * TILE + (c * CH + ((2 * w + g) ^ (c & 7))) * 16);
            f32x4 ka[2], tka[2];
            ka[0] = lds_read_f32x4(lk[0]);
            if constexpr (KV_TANGENT) tka[0] = lds_read_f32x4(lk[0] + (T_TK - T_K) * TILE);
#pragma unroll
            for (int u = 0; u < D / 8; ++u) {
                if (u + 1 < D / 8) {
                    const uint32_t at = lk[(u + 1) & 3] + 128 * ((u + 1) >> 2);
                    ka[(u + 1) & 1] = lds_read_f32x4(at);
                    if constexpr (KV_TANGENT) tka[(u + 1) & 1] = lds_read_f32x4(at + (T_TK - T_K) * TILE);
                }
                if (has_next) {                      // one 1-KiB part per wave and step
                    if (u >= 1 && u <= PT) stage_part(K, j0 + BC, nxt, T_K, u - 1);
                    if constexpr (KV_TANGENT)
                        if (u > PT && u <= 2 * PT) stage_part(tK, j0 + BC, nxt, T_TK, u - PT - 1);
                }
                FENCE();
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s = mfma32(ka[u & 1][e], q[u][e], s);
                    if constexpr (TANGENT) ts = mfma32(ka[u & 1][e], tq[u][e], ts);
                    if constexpr (KV_TANGENT) ts2 = mfma32(tka[u & 1][e], q[u][e], ts2);
                }
                FENCE();
            }
            asm volatile("" : "+v"(s));              // the vector ALU reads them: in arithmetic registers
            if constexpr (TANGENT) asm volatile("" : "+v"(ts));
            if constexpr (KV_TANGENT) {
                asm volatile("" : "+v"(ts2));
                ts += ts2;
            }
        }
        // ---- online softmax on this lane's 16 keys: register e holds key j0 + 8(e/4) + 4g + e%4
        const bool ragged = j0 + BC > Lkv;
        float mb = -INFINITY;
#pragma unroll
        for (int e = 0; e < 16; ++e) mb = fmaxf(mb, ragged && j0 + 8 * (e / 4) + 4 * g + (e % 4) >= Lkv ? -INFINITY : s[e] * scale);
        mb = xhalf_max(mb);
        const float m_new = mb > m + FP32_SLACK ? mb : m;
        const float alpha = m_new == m ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * LOG2E);    // 0 on the first block (m = -inf), else 1 or tiny
        m = m_new;
        const float m_ref = m == -INFINITY ? 0.f : m;       // (scores of -inf only so far, e.g. all of a part's: weight 0, not NaN)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0, 0)) {
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                asm volatile("" : "+a"(acc_o[n]));
                acc_o[n] *= alpha;
                asm volatile("" : "+a"(acc_o[n]));
                if constexpr (TANGENT) {
                    asm volatile("" : "+a"(acc_t[n]));
                    acc_t[n] *= alpha;
                    asm volatile("" : "+a"(acc_t[n]));
                }
            }
        }
        float p[16], h[16], row_p = 0.f, row_h = 0.f;
        auto weigh = [&](auto E) __attribute__((always_inline)) {
            constexpr int e = decltype(E)::value;
            const bool dead = ragged && j0 + 8 * (e / 4) + 4 * g + (e % 4) >= Lkv;
            p[e] = dead ? 0.f : __builtin_amdgcn_exp2f(fmaf(s[e], scale, -m_ref) * LOG2E);
            row_p += p[e];
            if constexpr (TANGENT) {
                h[e] = dead ? 0.f : p[e] * (ts[e] * scale);
                row_h += h[e];
            }
        };
        // ---- O^T += V^T P~^T, (A+B)^T += V^T H~^T + tV^T P~^T; the next block's V, tV travel meanwhile
        {
            uint32_t lv[4];                          // key row 8 (t/4) + 4g + t%4, column 32n + c at chunk ^ (row & 7)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                lv[i] = lds0 + (uint32_t)((cur * NT + T_V) * TILE + (4 * g + i) * (D * 4) + (((c >> 2) ^ (4 * g + i)) << 4) + 4 * (c & 3));
            constexpr int TV_OFF = (T_TV - T_V) * TILE;
            float va[2][NC], tva[2][NC];
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                va[0][n] = lds_read_f32(lv[0] + 128 * n);
                if constexpr (KV_TANGENT) tva[0][n] = lds_read_f32(lv[0] + 128 * n + TV_OFF);
            }
            weigh(std::integral_constant<int, 0>{});
            static_for<16>([&](auto Tt) {
                constexpr int t = decltype(Tt)::value;
                if constexpr (t + 1 < 16) {
#pragma unroll
                    for (int n = 0; n < NC; ++n) {
                        const uint32_t at = lv[(t + 1) & 3] + 8 * ((t + 1) >> 2) * (D * 4) + 128 * n;
                        va[(t + 1) & 1][n] = lds_read_f32(at);
                        if constexpr (KV_TANGENT) tva[(t + 1) & 1][n] = lds_read_f32(at + TV_OFF);
                    }
                }
                if (has_next) {
                    if (t >= 1 && t <= PT) stage_part(V, j0 + BC, nxt, T_V, t - 1);
                    if constexpr (KV_TANGENT)
                        if (t > PT && t <= 2 * PT) stage_part(tV, j0 + BC, nxt, T_TV, t - PT - 1);
                }
                FENCE();
#pragma unroll
                for (int n = 0; n < NC; ++n) acc_o[n] = mfma32(va[t & 1][n], p[t], acc_o[n]);
                if constexpr (TANGENT) {
#pragma unroll
                    for (int n = 0; n < NC; ++n) acc_t[n] = mfma32(va[t & 1][n], h[t], acc_t[n]);
                }
                if constexpr (KV_TANGENT) {
#pragma unroll
                    for (int n = 0; n < NC; ++n) acc_t[n] = mfma32(tva[t & 1][n], p[t], acc_t[n]);
                }
                if constexpr (t + 1 < 16) weigh(std::integral_constant<int, t + 1>{});
                FENCE();
            });
        }
        l = fmaf(alpha, l, row_p);
        r = fmaf(alpha, r, row_h);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wave's share of the next stage has landed
        __syncthreads();     // next stage written by all, this stage read by all
    }
}

// PARTS: keys in parts, an instantiation of its own (its bookkeeping in the one for whole calls cost those of few blocks: fp32 d64
// without tangents, H8 L2668, 98.4 -> 101.1 us; d128, query tangents, H20 Lq1700 Lkv77 52.5 -> 53.2).
template <int D, int TAN, bool PARTS>
__global__ __launch_bounds__(NTHREADS, (Geo<D, TAN>::WG_PER_CU)) void attn_jvp_mfma_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ tQ, const float* __restrict__ tK, const float* __restrict__ tV,
    float* __restrict__ O, float* __restrict__ tO, float* __restrict__ LSE,
    int Lq, int keys, float scale, int q_tiles, int H, int blhd, int parts_in, int part_blocks, f32x4* __restrict__ part_state) {
    // No implicit fusing of a product with a following sum: the compiler would fuse differently in each instantiation,
    // and the instantiations must agree bit for bit (absent tangents against zero tangents).  fmaf() stays fused.
#pragma clang fp contract(off)
    using G = Geo<D, TAN>;
    constexpr bool TANGENT = TAN != TAN_NONE, KV_TANGENT = TAN == TAN_ALL;
    constexpr int NT = D / 16;                       // score steps
    constexpr int NC = D / 32;                       // 32-column blocks of the accumulators
    constexpr int NX = KV_TANGENT ? 2 : 1;           // tensors on each of the K and V sides
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, g = lane >> 5;

    // consecutive workgroups go round-robin over the 8 XCDs: give each XCD a contiguous range of tiles, so that the
    // workgroups sharing one L2 stream the same heads' keys
    const int n_wg = gridDim.x;
    const int bid = (n_wg & 7) == 0 ? (int)(blockIdx.x & 7) * (n_wg >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    // (keys in parts, see attn_jvp_split.hip: a tile's K and V are those of its part, its results row bhp Lq + query of the
    // partial states)
    const int parts = PARTS ? parts_in : 1;
    const long bhp = bid / q_tiles;
    const long bh = parts > 1 ? bhp / parts : bhp;
    const int key0 = parts > 1 ? (int)(bhp - bh * parts) * part_blocks * BC : 0;
    const int Lkv = parts > 1 && keys - key0 > part_blocks * BC ? part_blocks * BC : keys - key0;
    const int qrow = (bid % q_tiles) * BR + 32 * wave + c;
    const int qload = qrow < Lq ? qrow : Lq - 1;     // rows past the end repeat the last one and are not stored

    // [B,H,L,d]: rows of a head contiguous; [B,L,H,d]: rows of a head H*d elements apart
    const long row_elems = blhd ? (long)H * D : D;
    const long bidx = bh / H, hidx = bh % H;
    const long q_base = blhd ? (bidx * Lq * H + hidx) * D : bh * (long)Lq * D;
    const long kv_base = (blhd ? (bidx * keys * H + hidx) * D : bh * (long)keys * D) + (long)key0 * row_elems;
    const int row_bytes = (int)(row_elems * sizeof(float));       // (32 rows are below 2^31 bytes: checked on the host)
    const int n_blocks = (Lkv + BC - 1) / BC;

    // ---- fetching a block into registers ----------------------------------------------------------------------------
    // K side: lane handles 8 consecutive elements (chunk k_sub) of row k_row (+ K_ROWS per pass).  V side: lane handles
    // one column of the 8 keys 16 (wave >> 1) + 4 (wave & 1) + {0..3, 8..11}: the keys of one 16-byte chunk.
    // Rows past the end of a ragged last block re-read rows inside it (finite values for finite inputs; their weight
    // is zero; those of V in turn, so that eight keys stay as many different ones as there are, or nearly), blocks past the end the
    // last block.
    // (No branches in here: lanes without a chunk or column of their own do their neighbour's once more, to the same place.)
    const int k_sub = tid % G::LPR < D / 8 ? tid % G::LPR : D / 8 - 1;
    const int k_row = tid / G::LPR < BC ? tid / G::LPR : tid / G::LPR - BC;
    const int v_key0 = 16 * (wave >> 1) + 4 * (wave & 1);
    const uint32_t k_off0 = (uint32_t)(32 * k_sub);              // chunk inside a row
    constexpr int LAST_COLS = D % 64 == 0 ? 64 : D % 64;         // columns of the last V pass
    const int v_lane_last = lane < LAST_COLS ? lane : LAST_COLS - 1;
    // byte offsets of the lane's rows from the block's first one; the same in all blocks but a ragged last one
    uint32_t k_rows[G::K_PASSES], v_rows[8];
    auto set_k_rows = [&](int blk) __attribute__((always_inline)) {
        const int left = Lkv - (blk < n_blocks ? blk : n_blocks - 1) * BC;
#pragma unroll
        for (int p = 0; p < G::K_PASSES; ++p) k_rows[p] = (k_row + p * G::K_ROWS < left ? (uint32_t)((k_row + p * G::K_ROWS) * row_bytes) : 0u) + k_off0;
    };
    auto set_v_rows = [&](int blk) __attribute__((always_inline)) {
        const int left = Lkv - (blk < n_blocks ? blk : n_blocks - 1) * BC;
        const int turn = (int)(0x80000000u >> __builtin_clz(left)) - 1;      // (a power of two up to left, less 1)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int key = v_key0 + (i & 3) + 8 * (i >> 2), row = key < left ? key : key & turn;
            v_rows[i] = (uint32_t)(row * row_bytes) + 4 * (uint32_t)lane;
        }
    };
    // The conversion jobs of a block are the K passes of K (and tK), then the V passes of V (and tV).  At most RING
    // jobs' data are in registers at a time: the end of a job requests the data of the RING-th job after it.
    constexpr int N_KJ = NX * G::K_PASSES, N_VJ = NX * G::V_PASSES, N_JOBS = N_KJ + N_VJ;
    constexpr int RING = N_JOBS < 4 ? N_JOBS : TAN == TAN_NONE && D >= 96 ? 2 : 4;      // (two workgroups share a unit there: fewer registers)
    static_assert(N_JOBS % RING == 0, "a job keeps its slot from block to block");
    float raw[RING][8];
    auto fetch_k = [&](int blk, auto J, float (&to)[8]) __attribute__((always_inline)) {
        constexpr int jb = decltype(J)::value, x = jb / G::K_PASSES, p = jb % G::K_PASSES;
        const char* base = reinterpret_cast<const char*>(x ? tK : K) + kv_base * 4 + (long)((blk < n_blocks ? blk : n_blocks - 1) * BC) * row_bytes;
        const f32x4 a = *reinterpret_cast<const f32x4*>(base + k_rows[p]), b = *reinterpret_cast<const f32x4*>(base + k_rows[p] + 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) { to[i] = a[i]; to[4 + i] = b[i]; }
    };
    auto fetch_v = [&](int blk, auto J, float (&to)[8]) __attribute__((always_inline)) {
        constexpr int jb = decltype(J)::value, x = (jb - N_KJ) / G::V_PASSES, p = (jb - N_KJ) % G::V_PASSES;
        const char* base = reinterpret_cast<const char*>(x ? tV : V) + kv_base * 4 + (long)((blk < n_blocks ? blk : n_blocks - 1) * BC) * row_bytes;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t at = 64 * (p + 1) <= D ? v_rows[i] : v_rows[i] + 4 * (uint32_t)(v_lane_last - lane);
            to[i] = *reinterpret_cast<const float*>(base + at + 256 * p);
        }
    };

    // ---- splitting what was fetched into the LDS planes, cut into parts for the MFMA shadows ------------------------
    const uint32_t k_write = lds0 + (uint32_t)(k_row * (2 * D) + ((k_sub ^ G::k_swizzle(k_row)) << 4));
    const uint32_t v_write = lds0 + G::V_BASE + (uint32_t)(lane * 64 + ((wave ^ ((lane >> 2) & 3)) << 4));
    const uint32_t v_write_last = lds0 + G::V_BASE + (uint32_t)(v_lane_last * 64 + ((wave ^ ((v_lane_last >> 2) & 3)) << 4));
    float v_scale[NX];                                   // set from the first block
    uint32_t v_low[NX], v_high[NX], v_ample;     // bits of 2^V_FLOOR, 2^16 and 2^6, scaled (v_low: less 1)
    uint64_t misfit = 0;         // lanes that have met values their tensor's scale does not suit
    int v_hits = 0;              // blocks in which values below it were met in this lane's columns,
    int v_hits_before = 0;       // ... but for the last one converted
    bool v_small[G::V_PASSES];   // is V of the block under way small or zero there?
    uint32_t cv_h[4], cv_l[4];
    float cv_mx, cv_m2, cv_sc, cv_own;
    uint64_t uneven[G::K_PASSES];        // lanes of the block under way that have met elements below their row's span
    // row factors: written by the first lane of a row (the others write to a place nobody reads: to one address their
    // writes would queue up)
    const uint32_t f_write = lds0 + (tid % G::LPR == 0 ? G::F_BASE + 4 * k_row : G::DUMMY_BASE + 4 * lane);
    // (the DPP steps of a row maximum one per part: the MFMA between two of them is the wait they need)
    constexpr int K_PARTS = 13, V_PARTS = 6;
    auto split_part = [&](const float (&e)[8], float s, auto PART) __attribute__((always_inline)) {      // parts 0-3
        constexpr int part = decltype(PART)::value, i = 2 * (part >> 1);
        if constexpr ((part & 1) == 0) { cv_h[i] = split_hi(e[2 * i], e[2 * i + 1], s); cv_h[i + 1] = split_hi(e[2 * i + 2], e[2 * i + 3], s); }
        else { cv_l[i] = split_lo(e[2 * i], e[2 * i + 1], s, cv_h[i]); cv_l[i + 1] = split_lo(e[2 * i + 2], e[2 * i + 3], s, cv_h[i + 1]); }
    };
    auto k_part = [&](auto J, auto ST, auto PART, const float (&e)[8]) __attribute__((always_inline)) {
        constexpr int jb = decltype(J)::value, x = jb / G::K_PASSES, p = jb % G::K_PASSES, st = decltype(ST)::value, part = decltype(PART)::value;
        if constexpr (part == 0) { cv_mx = max_abs3(e[0], e[1], e[2]); cv_m2 = max_abs3(e[3], e[4], e[5]); }
        if constexpr (part == 1) cv_mx = max_abs3(cv_mx, e[6], e[7]);
        if constexpr (part == 2) cv_mx = max_abs3(cv_mx, cv_m2, cv_m2);
        if constexpr (part == 3) cv_own = cv_mx;
        if constexpr (part == 3) cv_mx = max_dpp<0xB1>(cv_mx);             // lanes ^ 1, ^ 2, mirrored in 8, mirrored in 16
        if constexpr (part == 4) cv_mx = max_dpp<0x4E>(cv_mx);
        if constexpr (part == 5 && G::LPR >= 8) cv_mx = max_dpp<0x141>(cv_mx);
        if constexpr (part == 6 && G::LPR >= 16) cv_mx = max_dpp<0x140>(cv_mx);
        if constexpr (part == 7) {
            const int ex = top_exponent(cv_mx);
            cv_sc = pow2(254 + ROW_TOP - ex);
            const float factor = pow2(ex - ROW_TOP);
            const uint64_t low = __builtin_amdgcn_ballot_w64(below_span(cv_own, factor));
            uneven[p] = x ? uneven[p] | low : low;
            lds_write_f32(f_write + (st * 2 + x) * (BC * 4) + 4 * p * G::K_ROWS, factor);
        }
        if constexpr (part >= 8 && part < 12) split_part(e, cv_sc, std::integral_constant<int, part - 8>{});
        if constexpr (part == 12) {
            const uint32_t at = k_write + st * G::STAGE + 2 * x * G::PLANE + p * G::K_ROWS * 2 * D;
            lds_write_b128(at, u32x4{cv_h[0], cv_h[1], cv_h[2], cv_h[3]});
            lds_write_b128(at + G::PLANE, u32x4{cv_l[0], cv_l[1], cv_l[2], cv_l[3]});
        }
    };
    // What the conversion of block blk has found, as a rule nothing, is noted for the next iteration, which weighs the block: its
    // uneven keys, and that the rest of the sweep is for nothing.  The iteration after that clears the keys (noted), two
    // before those of block blk + 4 may be noted in the same place.
    const uint32_t note_base = lds0 + G::NOTE_BASE;
    if (tid < 8) lds_write_f32(note_base + 4 * tid, 0.f);
    auto write_note = [&](int blk) __attribute__((always_inline)) {
        uint64_t any = misfit;
#pragma unroll
        for (int p = 0; p < G::K_PASSES; ++p) any |= uneven[p];
        if (__builtin_expect(any != 0, 0)) {
            typedef __attribute__((address_space(3))) uint32_t lds_u32;
            uint32_t row = k_row;
            asm volatile("" : "+v"(row));
            lds_u32* note = reinterpret_cast<lds_u32*>((uintptr_t)(note_base + 8 * (blk & 3)));
#pragma unroll
            for (int p = 0; p < G::K_PASSES; ++p)
                if (uneven[p] >> lane & 1) __hip_atomic_fetch_or(note, 1u << (row + p * G::K_ROWS), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (misfit != 0) note[1] = 1;
        }
    };
    auto v_part = [&](auto J, auto ST, auto PART, const float (&e)[8]) __attribute__((always_inline)) {
        constexpr int jb = decltype(J)::value, x = (jb - N_KJ) / G::V_PASSES, p = (jb - N_KJ) % G::V_PASSES;
        constexpr int st = decltype(ST)::value, part = decltype(PART)::value;
        if constexpr (part == 0) {                       // do the eight values, one column of eight keys, suit the scale?
            const uint32_t top = __float_as_uint(max_abs3(max_abs3(max_abs3(max_abs3(e[0], e[1], e[2]), e[3], e[4]), e[5], e[6]), e[7], e[7]));
            misfit |= __builtin_amdgcn_ballot_w64(top >= v_high[x]);
            bool low = top - 1 < v_low[x];               // (a zero wraps around)
            if constexpr (x == 1) low &= v_small[p];
            else if constexpr (KV_TANGENT) v_small[p] = top < v_ample;
            v_hits += low ? 1 : 0;
        }
        if constexpr (part >= 1 && part < 5) split_part(e, v_scale[x], std::integral_constant<int, part - 1>{});
        if constexpr (part == 5) {
            const uint32_t at = (64 * (p + 1) <= D ? v_write : v_write_last) + st * G::STAGE + 2 * x * G::PLANE + p * 4096;
            lds_write_b128(at, u32x4{cv_h[0], cv_h[1], cv_h[2], cv_h[3]});
            lds_write_b128(at + G::PLANE, u32x4{cv_l[0], cv_l[1], cv_l[2], cv_l[3]});
        }
    };
    // The conversion of one block as a flat list of parts.  The last part of a job requests the RING-th job after it: of
    // the same blocks (bk on the K side, bv on the V side) or of the next.
    constexpr int N_PARTS = N_KJ * K_PARTS + N_VJ * V_PARTS;
    auto fetch_job = [&](auto J, int bk, int bv) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        if constexpr (j < N_KJ) fetch_k(bk, J, raw[j % RING]);
        else fetch_v(bv, J, raw[j % RING]);
    };
    // block whose V an iteration requests, from the one it converts: its own if the ring is shorter than the list
    constexpr int V_AHEAD = N_JOBS > RING ? 0 : 1;
    auto fetch_ahead = [&](auto J, int bk, int bv) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value + RING;
        if constexpr (j < N_JOBS) fetch_job(std::integral_constant<int, j>{}, bk, bv);
        else fetch_job(std::integral_constant<int, j - N_JOBS>{}, bk + 1, bv + 1);
    };
    auto convert_part = [&](auto IDX, auto KST, auto VST, int bk, int bv) __attribute__((always_inline)) {
        constexpr int idx = decltype(IDX)::value;
        if constexpr (idx < N_KJ * K_PARTS) {
            using J = std::integral_constant<int, idx / K_PARTS>;
            k_part(J{}, KST, std::integral_constant<int, idx % K_PARTS>{}, raw[J::value % RING]);
            if constexpr (idx % K_PARTS == K_PARTS - 1) fetch_ahead(J{}, bk, bv);
        } else {
            constexpr int r = idx - N_KJ * K_PARTS;
            using J = std::integral_constant<int, N_KJ + r / V_PARTS>;
            v_part(J{}, VST, std::integral_constant<int, r % V_PARTS>{}, raw[J::value % RING]);
            if constexpr (r % V_PARTS == V_PARTS - 1) fetch_ahead(J{}, bk, bv);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    // ---- this lane's query row, columns 16 t + 8 g .. + 7, split; a negative scale goes into the signs --------------
    const float sgn = scale < 0.f ? -1.f : 1.f;
    const float abs_scale = fabsf(scale);
    u32x4 qh[NT], ql[NT], tqh[TANGENT ? NT : 1], tql[TANGENT ? NT : 1];
    float fq = 1.f, ftq = 1.f;                       // what the scaled rows have to be multiplied by
    static_assert(RING >= N_KJ && RING >= N_VJ, "the jobs of either side fit the ring");
    set_k_rows(0);
    set_v_rows(0);
    // everything the prologue needs is requested at once: K(0), this lane's query row (below), V(0), K(1)
    float k0[N_KJ][8], k1[N_KJ][8], v0[N_VJ][8];
    static_for<N_KJ>([&](auto J) { fetch_k(0, J, k0[decltype(J)::value]); });
    float4 qraw[NT][2], tqraw[TANGENT ? NT : 1][2];
    auto fetch_query = [&](const float* X, float4 (*a)[2]) __attribute__((always_inline)) {
        const float* p = X + q_base + (long)qload * row_elems + 8 * g;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            a[t][0] = *reinterpret_cast<const float4*>(p + 16 * t);
            a[t][1] = *reinterpret_cast<const float4*>(p + 16 * t + 4);
        }
    };
    fetch_query(Q, qraw);
    if constexpr (TANGENT) fetch_query(tQ, tqraw);
    static_for<N_VJ>([&](auto J) { fetch_v(0, std::integral_constant<int, N_KJ + decltype(J)::value>{}, v0[decltype(J)::value]); });
    set_k_rows(1);
    static_for<N_KJ>([&](auto J) { fetch_k(1, J, k1[decltype(J)::value]); });
    FENCE();
    auto split_query = [&](const float4 (*a)[2], u32x4* hi, u32x4* lo, float& f) __attribute__((always_inline)) {
        float own[NT], mx = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 a0 = a[t][0], a1 = a[t][1];
            own[t] = max_abs3(max_abs3(a0.x, a0.y, a0.z), max_abs3(a0.w, a1.x, a1.y), max_abs3(a1.z, a1.w, a1.w));
            mx = fmaxf(mx, own[t]);
        }
        mx = xhalf_max(mx);
        const int ex = top_exponent(mx);
        const float s = sgn * pow2(254 + ROW_TOP - ex);
        f = pow2(ex - ROW_TOP);
        bool low = false;
#pragma unroll
        for (int t = 0; t < NT; ++t) low |= below_span(own[t], f);
        misfit |= __builtin_amdgcn_ballot_w64(low);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float e[8] = {a[t][0].x, a[t][0].y, a[t][0].z, a[t][0].w, a[t][1].x, a[t][1].y, a[t][1].z, a[t][1].w};
            static_for<4>([&](auto PART) { split_part(e, s, PART); });
            hi[t] = u32x4{cv_h[0], cv_h[1], cv_h[2], cv_h[3]};
            lo[t] = u32x4{cv_l[0], cv_l[1], cv_l[2], cv_l[3]};
            asm volatile("" : "+a"(hi[t]), "+a"(lo[t]));      // only MFMAs read them: keep them in accumulation registers
        }
        FENCE();
    };
    split_query(qraw, qh, ql, fq);
    if constexpr (TANGENT) split_query(tqraw, tqh, tql, ftq);
    // per-lane factor of the scores (after the key's own); not zero, so that masked scores stay -inf
    const float sq = fmaxf(abs_scale, 1e-37f) * fq;

    // ---- scores ----------------------------------------------------------------------------------------------------
    uint32_t kaddr[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) kaddr[t] = lds0 + c * (2 * D) + (((2 * t + g) ^ G::k_swizzle(c)) << 4);
    uint32_t vaddr[2];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) vaddr[t2] = lds0 + G::V_BASE + c * 64 + (((2 * t2 + g) ^ ((c >> 2) & 3)) << 4);
    const uint32_t faddr = lds0 + G::F_BASE + 16 * g;         // register e holds key 8 (e / 4) + 4 g + e % 4

    f32x16 s, ts1, ts2;      // K Q^T, K tQ^T, tK Q^T of the block under way (scaled; see `prepare` for the factors)
    // one score step: 3, 6 or 9 products; small terms first.  `behind(k)` is issued behind product number k of the block.
    constexpr int NS = KV_TANGENT ? 9 : TANGENT ? 6 : 3;
    constexpr int M1 = NT * NS;
    // Fragments X, tX: the high planes of the current and the next step, the low planes of the current one, which are
    // used by the first third of a step's products and then make room for the next step's
    u32x4 fh[2][NX], fl[NX];
    auto read_k = [&](auto T, auto ST, auto LO) __attribute__((always_inline)) {
        constexpr int t = decltype(T)::value, st = decltype(ST)::value;
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const uint32_t at = kaddr[t] + st * G::STAGE + 2 * x * G::PLANE;
            if constexpr (decltype(LO)::value) fl[x] = lds_read_b128(at + G::PLANE);
            else fh[t & 1][x] = lds_read_b128(at);
        }
    };
    auto scores = [&](auto ST, auto&& behind, auto&& first_values) __attribute__((always_inline)) {
        read_k(I0{}, ST, I1{});
        read_k(I0{}, ST, I0{});
        static_for<NT>([&](auto T) {
            constexpr int t = decltype(T)::value;
            using Tn = std::integral_constant<int, t + 1 < NT ? t + 1 : t>;
            if constexpr (t + 1 < NT) read_k(Tn{}, ST, I0{});
            else first_values(I0{});      // (the value products' first fragments, into the registers that are free)
            static_for<3>([&](auto W) {                      // lo hi, hi lo, hi hi
                constexpr int w = decltype(W)::value;
                constexpr int k0 = t * NS + w * (NS / 3);
                const u32x4 kh = fh[t & 1][0], kl = fl[0];
                if constexpr (w == 1 && t + 1 < NT) read_k(Tn{}, ST, I1{});
                if constexpr (w == 1 && t + 1 == NT) first_values(I1{});
                FENCE();
                if constexpr (t == 0 && w == 0) SMFMA0(kl, qh[t], s);
                else if constexpr (w == 0) SMFMA(kl, qh[t], s);
                else if constexpr (w == 1) SMFMA(kh, ql[t], s);
                else SMFMA(kh, qh[t], s);
                behind(std::integral_constant<int, k0>{});
                if constexpr (TANGENT) {
                    FENCE();
                    if constexpr (t == 0 && w == 0) SMFMA0(kl, tqh[t], ts1);
                    else if constexpr (w == 0) SMFMA(kl, tqh[t], ts1);
                    else if constexpr (w == 1) SMFMA(kh, tql[t], ts1);
                    else SMFMA(kh, tqh[t], ts1);
                    behind(std::integral_constant<int, k0 + 1>{});
                }
                if constexpr (KV_TANGENT) {
                    const u32x4 tkh = fh[t & 1][NX - 1], tkl = fl[NX - 1];
                    FENCE();
                    if constexpr (t == 0 && w == 0) SMFMA0(tkl, qh[t], ts2);
                    else if constexpr (w == 0) SMFMA(tkl, qh[t], ts2);
                    else if constexpr (w == 1) SMFMA(tkh, ql[t], ts2);
                    else SMFMA(tkh, qh[t], ts2);
                    behind(std::integral_constant<int, k0 + 2>{});
                }
                FENCE();
            });
        });
        SCORE_RESULTS_LAND();
        FENCE();
        asm volatile("" : "+v"(s));
        if constexpr (TANGENT) asm volatile("" : "+v"(ts1));
        if constexpr (KV_TANGENT) asm volatile("" : "+v"(ts2));
        FENCE();
    };

    // ---- softmax of one block: prepare (key factors, row maximum, reference), then the weights pair by pair ----------
    float m = -INFINITY;                             // row reference in nats: P~ = exp(S - m)
    float l = 0.f, r = 0.f;      // this lane's 16 keys per block only; halves meet in the epilogue
    float fqh = 0.f, ftqh = 0.f;                     // per-lane factors of the tangent scores, with 2^-eH
    float go = 1.f, gt = 1.f, gr = 1.f / P_GAIN;                        // factors of the accumulators
    float alpha = 1.f;
    bool moved = false;
    float w_uneven = 0.f;        // this lane's weights on uneven keys
    f32x2 note;                  // of the block under way
    bool noted = false;          // the last block's note is to be cleared
    f32x16 acc_o[NC], acc_t[TANGENT ? NC : 1];
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        acc_o[n] = f32x16{};
        if constexpr (TANGENT) acc_t[n] = f32x16{};
    }
    // (no instruction: keeps the accumulators in the accumulation registers across the score products, whose operands and
    // results need the arithmetic ones)
    auto pin_accumulators = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NC; ++n) {
            asm volatile("" : "+a"(acc_o[n]));
            if constexpr (TANGENT) asm volatile("" : "+a"(acc_t[n]));
        }
    };
    // key factors by quarters of the block (registers 4 q .. + 3), requested three quarters ahead of their use (two where
    // registers are shortest: D = 128 without tangents 867 -> 843 us on B2 H16 L4096)
    constexpr int KF = TAN == TAN_NONE && D == 128 ? 2 : 3;
    f32x4 kf[KF];
    auto read_factors = [&](auto Qi, auto ST) __attribute__((always_inline)) {
        constexpr int qi = decltype(Qi)::value;
        if constexpr (qi < 4) kf[qi % KF] = lds_read_f32x4(faddr + decltype(ST)::value * (2 * BC * 4) + 32 * qi);
    };
    auto key_factors = [&](auto E2, auto ST) __attribute__((always_inline)) {     // registers 2 E2, 2 E2 + 1
        constexpr int e0 = 2 * decltype(E2)::value, qi = e0 / 4;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            s[e0 + i] *= kf[qi % KF][e0 % 4 + i];
            if constexpr (TANGENT) ts1[e0 + i] *= kf[qi % KF][e0 % 4 + i];
        }
        if constexpr (e0 % 4 == 2) read_factors(std::integral_constant<int, qi + KF>{}, ST);
    };
    auto mask_tail = [&](int blk) __attribute__((always_inline)) {         // keys past the end weigh nothing
        const int jb = blk * BC + 4 * g;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (jb + 8 * (e / 4) + (e % 4) >= Lkv) {
                s[e] = -INFINITY;
                if constexpr (TANGENT) ts1[e] = 0.f;
                if constexpr (KV_TANGENT) ts2[e] = 0.f;
            }
    };
    auto row_max = [&]() __attribute__((always_inline)) -> float {
        const float a = max3(max3(s[0], s[1], s[2]), max3(s[3], s[4], s[5]), max3(s[6], s[7], s[8]));
        const float b = max3(max3(s[9], s[10], s[11]), max3(s[12], s[13], s[14]), s[15]);
        return xhalf_max(fmaxf(a, b));
    };
    auto follow_max = [&](float mx) __attribute__((always_inline)) {       // Alg. 2's rescale, when a row needs it
        const float mb = mx * sq;
        const bool up = mb > m + P_SLACK;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(up) != 0, 0)) {
            const float m_new = up ? mb : m;
            alpha = __builtin_amdgcn_exp2f((m - m_new) * LOG2E);
            m = m_new;
            l *= alpha; r *= alpha; w_uneven *= alpha;
            moved = true;
        }
    };
    auto rescale = [&]() __attribute__((always_inline)) {
        if (__builtin_expect(moved, 0)) {
            // (the empty statements tie the accumulators to the accumulation registers on entry and exit, so that the
            // copies to and from arithmetic registers stay inside this block)
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                asm volatile("" : "+a"(acc_o[n]));
                acc_o[n] *= alpha;
                asm volatile("" : "+a"(acc_o[n]));
                if constexpr (TANGENT) {
                    asm volatile("" : "+a"(acc_t[n]));
                    acc_t[n] *= alpha;
                    asm volatile("" : "+a"(acc_t[n]));
                }
            }
            moved = false;
        }
    };
    uint32_t ph[8], pl[8], hh[TANGENT ? 8 : 1], hl[TANGENT ? 8 : 1];        // split weights of the block under way ...
    uint32_t nph[4], npl[4], nhh[4], nhl[4];         // ... and of the next: its pairs 4-7, while this block's are still needed
    float p0, p1, h0, h1, u0, u1, x0, x1;
    float lb = 0.f, rb = 0.f;                        // sums over the block, added to l, r at its end
    constexpr int W_PARTS = TANGENT ? 8 : 4;
    auto weight_part = [&](auto J, auto ST, auto PART) __attribute__((always_inline)) {      // registers 2 J, 2 J + 1
        constexpr int j = decltype(J)::value, e = 2 * j, part = decltype(PART)::value;
        constexpr bool waits = j >= 4;
        uint32_t &wph = waits ? nph[j & 3] : ph[j], &wpl = waits ? npl[j & 3] : pl[j];
        uint32_t &whh = waits ? nhh[j & 3] : hh[TANGENT ? j : 0], &whl = waits ? nhl[j & 3] : hl[TANGENT ? j : 0];
        const float one = 1.f, gain = P_GAIN;
        if constexpr (part == 0) {
            x0 = fmaf(s[e], sq, -m) * LOG2E; x1 = fmaf(s[e + 1], sq, -m) * LOG2E;
            if constexpr (KV_TANGENT) {                      // (used by part 4)
                const f32x2 f = lds_read_f32x2(faddr + decltype(ST)::value * (2 * BC * 4) + BC * 4 + 32 * (e / 4) + 4 * (e % 4));
                u0 = f[0]; u1 = f[1];
            }
        }
        if constexpr (part == 1) { p0 = __builtin_amdgcn_exp2f(x0); p1 = __builtin_amdgcn_exp2f(x1); }
        if constexpr (part == 2) {
            lb = j == 4 ? p0 + p1 : lb + (p0 + p1);
            if (j == 3) l += lb;
            wph = split_hi(p0, p1, gain);
        }
        // (the empty statements hold the packing here, behind a product: its results are used by the next iteration or by the last
        // block's products, and the compiler would move it in front of either)
        if constexpr (part == 3) { wpl = split_lo(p0, p1, gain, wph); if constexpr (G::LAST_ALONE) asm volatile("" : "+v"(wpl)); }
        if constexpr (TANGENT) {
            if constexpr (part == 4) {
                if constexpr (KV_TANGENT) { u0 = (ts2[e] * u0) * fqh; u1 = (ts2[e + 1] * u1) * fqh; }
            }
            if constexpr (part == 5) {
                if constexpr (KV_TANGENT) { u0 = fmaf(ts1[e], ftqh, u0); u1 = fmaf(ts1[e + 1], ftqh, u1); }
                else { u0 = ts1[e] * ftqh; u1 = ts1[e + 1] * ftqh; }
                h0 = p0 * u0; h1 = p1 * u1;
            }
            if constexpr (part == 6) {
                rb = j == 4 ? h0 + h1 : rb + (h0 + h1);
                if (j == 3) r += rb;
                whh = pack_f16(h0, h1);
            }
            if constexpr (part == 7) { whl = split_lo(h0, h1, one, whh); if constexpr (G::LAST_ALONE) asm volatile("" : "+v"(whl)); }
        }
    };
    auto next_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ph[4 + i] = nph[i]; pl[4 + i] = npl[i];
            if constexpr (TANGENT) { hh[4 + i] = nhh[i]; hl[4 + i] = nhl[i]; }
        }
    };
    // Weights of the uneven keys of a block, from the high terms of the split ones: pairs 0-3 in ph, 4-7 still in nph.  Such a
    // key's score may lack up to 2^-25 of each of its scaled elements times the query's (2^13 at most), and its weight that
    // many nats: UNEVEN_SHARE leaves room for eight of them (a weight of zero is below 2^-37 of the row's reference), and
    // where there may be more the tile is redone.  Keys that a channel masks weigh zero and cost nothing.
    auto weigh_uneven = [&](uint32_t keys, uint32_t factors) __attribute__((always_inline)) {
        uint32_t mine = keys >> (4 * g);
        float most = 0.f;
        asm volatile("" : "+v"(mine), "+v"(factors));        // (nothing of this is computed ahead: registers are short)
        static_for<16>([&](auto E) {
            constexpr int e = decltype(E)::value, key = 8 * (e / 4) + e % 4;
            FENCE();
            const f16x2 w = __builtin_bit_cast(f16x2, e < 8 ? ph[e / 2] : nph[e / 2 & 3]);
            const float f = lds_read_f32(factors + 32 * (e / 4) + 4 * (e % 4));
            w_uneven += mine & 1u << key ? (float)w[e & 1] : 0.f;
            most = fmaxf(most, mine & 1u << key ? f : 0.f);
        });
        FENCE();
        if (most * sq * (D * 0x1p-12f) > 8.f) w_uneven = INFINITY;
    };
    auto read_note = [&](int blk) __attribute__((always_inline)) { note = lds_read_f32x2(note_base + 8 * (blk & 3)); };
    auto heed_note = [&](int blk) __attribute__((always_inline)) -> bool {      // true: the sweep is to end
        const uint32_t keys = __float_as_uint(note[0]), stop = __float_as_uint(note[1]);
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(keys | stop) == 0, 1)) return false;
        weigh_uneven(keys, faddr + (blk & 1) * (2 * BC * 4));
        noted = true;
        return __builtin_amdgcn_readfirstlane(stop) != 0;
    };
    // the softmax of a block as a flat list: key factors by pairs, the row maximum, pairs 4-7, then pairs 0-3 (whose
    // registers the first half of the value products has read by the time the list gets there: see the assertion below)
    constexpr int S_PRE = 10, S_PARTS = S_PRE + 8 * W_PARTS;
    float mx_row, top_row;       // a row's largest score in the block, and so far
    auto softmax_part = [&](auto IDX, auto ST, int blk) __attribute__((always_inline)) {
        constexpr int idx = decltype(IDX)::value;
        if constexpr (idx == S_PARTS - 4) read_note(blk);
        if constexpr (idx < 8) key_factors(IDX, ST);
        else if constexpr (idx == 8) {
            if ((blk + 1) * BC > Lkv) mask_tail(blk);
            mx_row = row_max();
        } else if constexpr (idx == 9) {
            follow_max(mx_row);
            top_row = fmaxf(top_row, mx_row);
        }
        if constexpr (idx >= S_PRE) weight_part(std::integral_constant<int, ((idx - S_PRE) / W_PARTS + 4) & 7>{}, ST, std::integral_constant<int, (idx - S_PRE) % W_PARTS>{});
    };

    // ---- value products of a block, small terms first ----------------------------------------------------------------
    constexpr int M2 = 2 * NC * NS;
    auto read_v = [&](auto Gi, auto ST, auto LO) __attribute__((always_inline)) {
        constexpr int gi = decltype(Gi)::value, t2 = gi / NC, n = gi % NC, st = decltype(ST)::value;
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const uint32_t at = vaddr[t2] + st * G::STAGE + 2 * x * G::PLANE + n * 2048;
            if constexpr (decltype(LO)::value) fl[x] = lds_read_b128(at + G::PLANE);
            else fh[gi & 1][x] = lds_read_b128(at);
        }
    };
    auto values = [&](auto&& read, auto&& behind) __attribute__((always_inline)) {      // read(Gi, LO): the fragments of group Gi; those of the first are there
        static_for<2 * NC>([&](auto Gi) {
            constexpr int gi = decltype(Gi)::value, t2 = gi / NC, n = gi % NC;
            using Gn = std::integral_constant<int, gi + 1 < 2 * NC ? gi + 1 : gi>;
            if constexpr (gi + 1 < 2 * NC) read(Gn{}, I0{});
            const u32x4 wph = {ph[4 * t2], ph[4 * t2 + 1], ph[4 * t2 + 2], ph[4 * t2 + 3]};
            const u32x4 wpl = {pl[4 * t2], pl[4 * t2 + 1], pl[4 * t2 + 2], pl[4 * t2 + 3]};
            u32x4 whh = wph, whl = wpl;
            if constexpr (TANGENT) {
                whh = u32x4{hh[4 * t2], hh[4 * t2 + 1], hh[4 * t2 + 2], hh[4 * t2 + 3]};
                whl = u32x4{hl[4 * t2], hl[4 * t2 + 1], hl[4 * t2 + 2], hl[4 * t2 + 3]};
            }
            static_for<3>([&](auto W) {                      // lo hi, hi lo, hi hi
                constexpr int w = decltype(W)::value;
                constexpr int k0 = gi * NS + w * (NS / 3);
                const u32x4 vh = fh[gi & 1][0], vl = fl[0];
                if constexpr (w == 1 && gi + 1 < 2 * NC) read(Gn{}, I1{});
                FENCE();
                acc_o[n] = mfma16(w == 0 ? vl : vh, w == 1 ? wpl : wph, acc_o[n]);
                behind(std::integral_constant<int, k0>{});
                if constexpr (TANGENT) {
                    FENCE();
                    acc_t[n] = mfma16(w == 0 ? vl : vh, w == 1 ? whl : whh, acc_t[n]);
                    behind(std::integral_constant<int, k0 + 1>{});
                }
                if constexpr (KV_TANGENT) {
                    const u32x4 tvh = fh[gi & 1][NX - 1], tvl = fl[NX - 1];
                    FENCE();
                    acc_t[n] = mfma16(w == 0 ? tvl : tvh, w == 1 ? wpl : wph, acc_t[n]);
                    behind(std::integral_constant<int, k0 + 2>{});
                }
                FENCE();
            });
        });
    };

    // ---- prologue: K(0), K(1), V(0) split, weights of block 0 --------------------------------------------------------
    auto nothing = [](auto) __attribute__((always_inline)) {};
    static_for<N_KJ * K_PARTS>([&](auto IDX) {
        constexpr int j = decltype(IDX)::value / K_PARTS;
        k_part(std::integral_constant<int, j>{}, I0{}, std::integral_constant<int, decltype(IDX)::value % K_PARTS>{}, k0[j]);
    });
    {
        float vm[2] = {0.f, 0.f};
        static_for<N_VJ>([&](auto J) {                   // largest |V|, |tV| of block 0
            constexpr int j = decltype(J)::value, x = j / G::V_PASSES;
#pragma unroll
            for (int i = 0; i < 8; i += 2) vm[x] = max_abs3(vm[x], v0[j][i], v0[j][i + 1]);
        });
        __syncthreads();                                 // K(0) and its row factors are in, the words of uneven keys cleared
        write_note(0);
        scores(I0{}, nothing, nothing);
        static_for<KF>([&](auto Qi) { read_factors(Qi, I0{}); });
        static_for<8>([&](auto E2) { key_factors(E2, I0{}); });
        if (BC > Lkv) mask_tail(0);
        top_row = row_max();
        m = top_row * sq;
        float t0 = 0.f;                                  // largest tangent score of the block, unscaled
        if constexpr (TANGENT) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float u = ts1[e] * (abs_scale * ftq);
                if constexpr (KV_TANGENT) u = fmaf(ts2[e] * lds_read_f32(faddr + BC * 4 + 32 * (e / 4) + 4 * (e % 4)), abs_scale * fq, u);
                t0 = max_abs3(t0, u, u);
            }
        }
        // largest of the workgroup; and the word of the vote at the end is cleared
        lds_write_f32(lds0 + G::RED_BASE + 48, 0.f);
        float red[3] = {vm[0], vm[1], t0};
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) red[i] = fmaxf(red[i], __shfl_xor(red[i], o));
            lds_write_f32(lds0 + G::RED_BASE + 4 * (4 * i + wave), red[i]);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const f32x4 w = lds_read_f32x4(lds0 + G::RED_BASE + 16 * i);
            red[i] = fmaxf(fmaxf(w[0], w[1]), fmaxf(w[2], w[3]));
        }
        // exponents; tV is scaled with V's factor times 2^-eH
        const int eV = top_exponent(red[0]) - 127 - V_TOP;
        int eH = 0;
        if constexpr (TANGENT) {
            eH = top_exponent(red[2]) - 127 + T_HEADROOM;
            const int rho = top_exponent(red[1]) - top_exponent(red[0]);
            eH = rho > eH ? rho : eH;
            const int lo = -100 - eV > -100 ? -100 - eV : -100, hi = 100 - eV < 100 ? 100 - eV : 100;
            eH = eH < lo ? lo : eH > hi ? hi : eH;           // every factor stays a normal number
        }
        go = ldexpf(1.f, eV - 12);
        gt = ldexpf(1.f, eV + eH - 12);
        v_scale[0] = ldexpf(1.f, -eV);
        if constexpr (KV_TANGENT) v_scale[1] = ldexpf(1.f, -(eV + eH));
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            const uint32_t one = (uint32_t)(eV + x * eH + 127) << 23;
            v_low[x] = __builtin_amdgcn_readfirstlane(one + (uint32_t)V_FLOOR * (1u << 23) - 1);
            v_high[x] = __builtin_amdgcn_readfirstlane(one < (239u << 23) ? one + (16u << 23) : 255u << 23);
        }
        v_ample = v_low[0] + V_AMPLE;
        ftqh = ldexpf(abs_scale * ftq, 12 - eH);
        fqh = ldexpf(abs_scale * fq, 12 - eH);
        static_for<8 * W_PARTS>([&](auto IDX) {
            weight_part(std::integral_constant<int, (decltype(IDX)::value / W_PARTS + 4) & 7>{}, I0{}, std::integral_constant<int, decltype(IDX)::value % W_PARTS>{});
        });
        // the first jobs of the sweep's first iteration: K(2), V(1); then V(0) -> stage 0, K(1) -> stage 1
        set_k_rows(2);
        set_v_rows(1);
        static_for<RING>([&](auto J) { fetch_job(J, 2, 1); });
        static_for<N_VJ * V_PARTS>([&](auto IDX) {
            constexpr int j = decltype(IDX)::value / V_PARTS;
            v_part(std::integral_constant<int, N_KJ + j>{}, I0{}, std::integral_constant<int, decltype(IDX)::value % V_PARTS>{}, v0[j]);
        });
        static_for<N_KJ * K_PARTS>([&](auto IDX) {
            constexpr int j = decltype(IDX)::value / K_PARTS;
            k_part(std::integral_constant<int, j>{}, I1{}, std::integral_constant<int, decltype(IDX)::value % K_PARTS>{}, k1[j]);
        });
        write_note(1);
        read_note(0);
        heed_note(0);
        __syncthreads();
    }

    // ---- sweep: iteration b does the scores of block b + 1 over the conversion of K(b + 2) and V(b + 1), then the values of
    // block b over the softmax of block b + 1.  Stage of a block: its index & 1.
    // (the last block, which may have few keys, counts twice: as the block past the end, or in the end)
    const int hits_enough = n_blocks + 1 < V_HITS ? n_blocks + 1 : V_HITS;
    auto iteration = [&](auto PAR, int b) __attribute__((always_inline)) -> bool {
        constexpr int par = decltype(PAR)::value;
        using Cur = std::integral_constant<int, par>;
        using Nxt = std::integral_constant<int, par ^ 1>;
        if constexpr (G::LAST_ALONE) v_hits_before = v_hits;
        next_weights();
        pin_accumulators();
        if (__builtin_expect(noted, 0)) {
            lds_write_f32(note_base + 8 * (b & 3), 0.f);
            noted = false;
        }
        if (__builtin_expect(b + 3 >= n_blocks - 1, 0)) {        // from here on requests may be for the last block
            set_k_rows(b + 3);
            set_v_rows(b + 1 + V_AHEAD);
        }
        scores(Nxt{}, [&](auto Kk) __attribute__((always_inline)) {
            constexpr int k = decltype(Kk)::value;
            constexpr int first = k * N_PARTS / M1, last = (k + 1) * N_PARTS / M1;
            static_for<last - first>([&](auto I) { convert_part(std::integral_constant<int, first + decltype(I)::value>{}, Cur{}, Nxt{}, b + 2, b + 1); });
        }, [&](auto LO) __attribute__((always_inline)) {
            read_v(I0{}, Cur{}, LO);
            if constexpr (decltype(LO)::value) static_for<KF>([&](auto Qi) { read_factors(Qi, Nxt{}); });
        });
        static_assert((S_PRE + 4 * W_PARTS) * M2 / S_PARTS >= M2 / 2, "pairs 0-3 come behind the second half of the value products");
        values([&](auto Gi, auto LO) __attribute__((always_inline)) { read_v(Gi, Cur{}, LO); }, [&](auto Kk) __attribute__((always_inline)) {
            constexpr int k = decltype(Kk)::value;
            constexpr int first = k * S_PARTS / M2, last = (k + 1) * S_PARTS / M2;
            static_for<last - first>([&](auto I) { softmax_part(std::integral_constant<int, first + decltype(I)::value>{}, Nxt{}, b + 1); });
        });
        rescale();
        if constexpr (TANGENT) misfit |= __builtin_amdgcn_ballot_w64(!(fabsf(rb) < 0x1p20f));      // sixteen H~ of fp16 size stay below
        misfit |= __builtin_amdgcn_ballot_w64(v_hits >= hits_enough);
        write_note(b + 2);
        const bool stop = heed_note(b + 1);
        __syncthreads();     // the next block's planes are written by all, this one's read by all
        return stop;
    };
    // (One loop body for all blocks, or all but the last: a copy of it for a tail made the register allocator move accumulators and operands
    // around.  The last block alone stands in straight-line code, from a stage by its index: behind a branch, left out where the sweep
    // was to end, it made the allocator spill 30 to 1200 bytes in the loop.  us a call, before -> now: all tangents H8 L700 d128 45.7 -> 43.4,
    // query tangents H20 Lq1700 Lkv77 d128 45.1 -> 42.3, B2 H24 Lq1500 Lkv128 d32 27.8 -> 23.7.)
    const int iterations = G::LAST_ALONE ? n_blocks - 1 : n_blocks;
    if (!G::LAST_ALONE || iterations > 0)
        for (int b = 0;;) {
            if (iteration(I0{}, b) || ++b >= iterations) break;
            if (iteration(I1{}, b) || ++b >= iterations) break;
        }
    if constexpr (G::LAST_ALONE) {
        next_weights();              // (for nothing if the sweep was to end)
        pin_accumulators();
        const uint32_t shift = (uint32_t)((n_blocks - 1) & 1) * G::STAGE;
        const uint32_t vlast[2] = {vaddr[0] + shift, vaddr[1] + shift};
        auto read_last = [&](auto Gi, auto LO) __attribute__((always_inline)) {
            constexpr int gi = decltype(Gi)::value, t2 = gi / NC, n = gi % NC;
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                const uint32_t at = vlast[t2] + 2 * x * G::PLANE + n * 2048;
                if constexpr (decltype(LO)::value) fl[x] = lds_read_b128(at + G::PLANE);
                else fh[gi & 1][x] = lds_read_b128(at);
            }
        };
        read_last(I0{}, I0{});
        read_last(I0{}, I1{});
        values(read_last, nothing);
        pin_accumulators();
        v_hits += v_hits - v_hits_before;
        misfit |= __builtin_amdgcn_ballot_w64(v_hits >= hits_enough);
    }

    // ---- did the scales suit?  If not, the workgroup redoes its tile ------------------------------------------------------
    // Too large: something is inf or NaN.  Too small: the lanes that converted V and tV have seen it (misfit), or a row's
    // results are small against what the fp16 terms resolve.  These are whole multiples of 2^-24: an accumulator is out by
    // 2^-25 of the V (2^9 as a rule, up to 2^12) of every key that counts for the rounding of its weight, and by up to
    // l 2^12 2^-25 for that of V or tV (which average out, unless all keys' are alike).  A row whose largest |O| or |A + B| is
    // 2^7 sqrt(l), and 2^2 l, knows it to 2^-24 sqrt(keys / l) or so for the one and 2^-15 at worst for the other.  Ordinary
    // rows (keys / l about 5, S of standard deviation 1) have |O| of 2^23 sqrt(l), |A + B| of 2^16 sqrt(l).
    // It takes weights on keys whose V is small beside the others', a sink without values for one, or tangent scores small
    // beside those of the tile's first block, to come near the line.  A row without tangents has exact zeros.  Where one key
    // has nearly all of a row's weight its tangent score alone makes A + B, which then is small by chance in one row of
    // hundreds; few keys count beside it, and A + B cancels against r O to its own rounding anyway: 2^-1 does there.
    auto too_small = [](float top, float l) __attribute__((always_inline)) { return top * top < ROW_FLOOR * l * fmaxf(l * 0x1p-10f, 1.f); };
    float bad = l * 0.f + r * 0.f;         // NaN once anything is inf or NaN
    float top_o = 0.f, top_t = 0.f;
#pragma unroll
    for (int n = 0; n < NC; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            bad = fmaf(acc_o[n][e], 0.f, bad);
            top_o = fmaxf(top_o, fabsf(acc_o[n][e]));
            if constexpr (TANGENT) {
                bad = fmaf(acc_t[n][e], 0.f, bad);
                top_t = fmaxf(top_t, fabsf(acc_t[n][e]));
            }
        }
    float l_row = xhalf_sum(l), r_row = xhalf_sum(r);
    top_o = xhalf_max(top_o);
    if (misfit != 0 || too_small(top_o, l_row) || !(xhalf_sum(w_uneven) <= l_row * (P_GAIN * UNEVEN_SHARE))) bad = 1.f;
    if constexpr (TANGENT) {
        top_t = xhalf_max(top_t);
        const bool one_key = l_row < ONE_KEY * __builtin_amdgcn_exp2f(fmaf(top_row, sq, -m) * LOG2E);
        if (too_small(one_key ? ONE_KEY_GAIN * top_t : top_t, l_row) && (r_row != 0.f || top_t != 0.f)) bad = 1.f;
    }
    if (__builtin_amdgcn_ballot_w64(bad != 0.f || bad != bad) != 0 && lane == 0) lds_write_f32(lds0 + G::RED_BASE + 48, 1.f);
    __syncthreads();
    const bool redo = __builtin_amdgcn_readfirstlane(__float_as_int(lds_read_f32(lds0 + G::RED_BASE + 48))) != 0;
    if (__builtin_expect(redo, 0)) {
        static_assert(2 * (KV_TANGENT ? 4 : 2) * BC * D * 4 <= G::F_BASE, "its stages fit, clear of the vote");
        go = 1.f; gt = 1.f; gr = 1.f;
        int here = lane, row = qload, w = wave;      // (nothing that it derives from these is kept across the sweep)
        asm volatile("" : "+v"(here), "+v"(row), "+s"(w));
        fp32_tile<D, TAN>(Q, K, V, tQ, tK, tV, q_base + (long)row * row_elems, kv_base, row_elems, Lkv, scale, lds0, here, w,
                          acc_o, acc_t, m, l_row, r_row);
        l_row = xhalf_sum(l_row);
        r_row = xhalf_sum(r_row);
    }

    // ---- epilogue (Alg. 2, last lines): accumulator register 4k + i of column block n is column 32n + 8k + 4g + i -----
    // A lane holds 16-byte pieces of one row, so stores from the registers move 32 bytes of each of 32 rows per instruction.  Each
    // wave turns its 32 rows round through its share of the idle stages (o and to in turn where there are no key tangents and
    // so half the stages), and stores whole rows, the reads for several stores in flight at once.  LDS operations of a
    // wave execute in order, so there is no barrier.  (us a call, before -> now: query tangents H20 Lq1700 Lkv77 d128 52.5 -> 45.1, B2 H16
    // Lq2048 Lkv512 d128 131.7 -> 123, all tangents H8 L700 d128 48.4 -> 45.7, H24 L3000 d32 486 -> 478.)
    {
        const float inv_l = 1.f / l_row;
        const float mu = r_row * inv_l * gr;         // rowsum(P o tS), in the accumulators' scale
        const float fo = go * inv_l, ft = gt * inv_l;
        int here = lane;                             // (nothing that is derived from it below is kept across the sweep)
        asm volatile("" : "+v"(here));
        constexpr bool DIRECT = D == 128 && !TANGENT;
        const int half = DIRECT ? g : here >> 5;
        if (half == 0 && qrow < Lq) {
            if constexpr (PARTS) part_state[bhp * Lq + qrow] = f32x4{m, l_row, mu * (gt / go), 0.f};
            else LSE[bh * Lq + qrow] = fmaf(__builtin_amdgcn_logf(l_row), LN2, m);     // v_log_f32 is a binary log
        }
        typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
        constexpr int ROW = D * 4, CHUNKS = D / 4, RPS = 64 / CHUNKS, N = 32 / RPS, BATCH = N < 8 ? N : 8;      // RPS: rows of a store
        static_assert(4 * 32 * ROW <= 4 * G::STAGE && (!KV_TANGENT || 8 * 32 * ROW <= 4 * G::STAGE), "the waves' shares fit the stages");
        auto swizzle = [](int row) { return D == 96 ? (row >> 1) & 7 : row & (CHUNKS - 1); };
        const uint32_t stage_o = lds0 + (uint32_t)wave * (32 * ROW), stage_t = KV_TANGENT ? stage_o + 4 * 32 * ROW : stage_o;
        const int q0 = __builtin_amdgcn_readfirstlane(qrow);
        const bool whole = q0 + 32 <= Lq;            // (uniform)
        auto turn = [&](uint32_t stage, auto&& value) __attribute__((always_inline)) {       // value(n, k): registers 4k .. + 3 of column block n
#pragma unroll
            for (int n = 0; n < NC; ++n)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *reinterpret_cast<lds_f32x4*>((uintptr_t)(stage + (uint32_t)(here & 31) * ROW + (uint32_t)(((8 * n + 2 * k + (here >> 5)) ^ swizzle(here & 31)) << 4))) = value(n, k);
        };
        auto store = [&](uint32_t stage, float* to) __attribute__((always_inline)) {
            const int piece = here % CHUNKS, r0 = here / CHUNKS;
            if (r0 >= RPS) return;                   // (head dimension 96: 48 lanes)
            const uint32_t lane_bytes = (uint32_t)r0 * (uint32_t)(PARTS ? ROW : 4 * row_elems) + 16 * piece;
#pragma unroll
            for (int i0 = 0; i0 < N; i0 += BATCH) {
                f32x4 x[BATCH];
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int r = RPS * (i0 + u) + r0;
                    x[u] = *reinterpret_cast<const lds_f32x4*>((uintptr_t)(stage + (uint32_t)r * ROW + (uint32_t)((piece ^ swizzle(r)) << 4)));
                }
                FENCE();
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int first = q0 + RPS * (i0 + u);
                    const long at = PARTS ? (bhp * Lq + first) * (long)D : q_base + (long)first * row_elems;
                    if (whole || first + r0 < Lq) {
                        f32x4* dst = reinterpret_cast<f32x4*>(reinterpret_cast<char*>(to + at) + lane_bytes);
                        if constexpr (PARTS) *dst = x[u];          // (the merge reads them next)
                        else __builtin_nontemporal_store(x[u], dst);
                    }
                }
                FENCE();
            }
        };
        auto value_o = [&](int n, int k) __attribute__((always_inline)) {
            return f32x4{acc_o[n][4 * k] * fo, acc_o[n][4 * k + 1] * fo, acc_o[n][4 * k + 2] * fo, acc_o[n][4 * k + 3] * fo};
        };
        auto value_t = [&](int n, int k) __attribute__((always_inline)) {
            return f32x4{fmaf(-mu, acc_o[n][4 * k], acc_t[n][4 * k]) * ft, fmaf(-mu, acc_o[n][4 * k + 1], acc_t[n][4 * k + 1]) * ft,
                         fmaf(-mu, acc_o[n][4 * k + 2], acc_t[n][4 * k + 2]) * ft, fmaf(-mu, acc_o[n][4 * k + 3], acc_t[n][4 * k + 3]) * ft};
        };
        if constexpr (DIRECT) {
            // (straight from the registers: those that the way through LDS needs were spilled in the sweep, and the other workgroup of
            // the unit covers these stores; B2 H16 L4096 846 us against 855)
            if (qrow < Lq) {
                float* op = O + (PARTS ? (bhp * Lq + qrow) * D : q_base + (long)qrow * row_elems) + 4 * half;
#pragma unroll
                for (int n = 0; n < NC; ++n)
#pragma unroll
                    for (int k = 0; k < 4; ++k) *reinterpret_cast<f32x4*>(op + 32 * n + 8 * k) = value_o(n, k);
            }
        } else {
            turn(stage_o, value_o);
            if constexpr (KV_TANGENT) turn(stage_t, value_t);
            store(stage_o, O);
            if constexpr (TANGENT) {
                if constexpr (!KV_TANGENT) turn(stage_t, value_t);
                store(stage_t, tO);
            }
        }
    }
}

template <int D, int TAN, bool PARTS>
hipError_t launch_parts(const Problem& p) {
    const int q_tiles = (p.Lq + BR - 1) / BR;
    const long long blocks = (long long)q_tiles * p.B * p.H * p.split.parts;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const PartStates ps = part_states(p);
    constexpr int smem = Geo<D, TAN>::LDS_BYTES;
    auto kern = attn_jvp_mfma_f32_kernel<D, TAN, PARTS>;
    int dev = 0, cus = 0;
    hipError_t e = device_cus(&dev, &cus);
    if (e == hipSuccess) e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, dev);
    if (e != hipSuccess) return e;
    MainKernelTimer timer(p);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(NTHREADS), smem, p.stream,
                       (const float*)p.q, (const float*)p.k, (const float*)p.v,
                       (const float*)p.tq, (const float*)p.tk, (const float*)p.tv,
                       (float*)ps.o, (float*)ps.to, p.lse, p.Lq, p.Lkv, p.scale, q_tiles, p.H, p.layout, p.split.parts, p.split.blocks,
                       (f32x4*)ps.state);
    e = hipGetLastError();
    if (e == hipSuccess && PARTS) e = launch_merge_parts(p, ps);
    return timer.finish(e);
}

template <int D, int TAN>
hipError_t launch_one(const Problem& p) {
    return p.split.parts > 1 ? launch_parts<D, TAN, true>(p) : launch_parts<D, TAN, false>(p);
}

template <int D>
hipError_t launch_tan(const Problem& p) {
    if (!p.tq) return launch_one<D, TAN_NONE>(p);
    if (!p.tk) return launch_one<D, TAN_QUERY>(p);
    return launch_one<D, TAN_ALL>(p);
}

}  // namespace

bool mfma_f32_supports(const Problem& p) {
    // (a lane's byte offset inside a block of 32 rows is kept in 32 bits)
    const long long row_bytes = (long long)(p.layout ? p.H : 1) * p.d * (long long)sizeof(float);
    return p.in_dtype == 1 && (p.d == 32 || p.d == 64 || p.d == 96 || p.d == 128) && row_bytes * BC < (1ll << 31);
}

hipError_t launch_mfma_f32(const Problem& p) {
    if (!mfma_f32_supports(p)) return hipErrorInvalidValue;
    switch (p.d) {
        case 32: return launch_tan<32>(p);
        case 64: return launch_tan<64>(p);
        case 96: return launch_tan<96>(p);
        default: return launch_tan<128>(p);
    }
}

}  // namespace attn_jvp
