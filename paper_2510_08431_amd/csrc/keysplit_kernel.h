// Attention forward + JVP (paper App. C.1, Alg. 2) with the KEYS dealt to the waves of a workgroup: head dimensions 32, 64,
// 96, 128 and 256, fp32 or bf16 inputs, fp32-accurate results.  For calls whose 128-row tiles would leave most of the chip
// idle, and for head dimension 256, whose accumulators do not fit a wave that owns 32 rows.
//
// A workgroup owns 16 query rows of a head; wave w of NW takes the key blocks w, w + NW, ... (32 keys each) through
// Alg. 2's loop by itself, with its own running reference, and the NW partial states (m, l, r, O~, A + B) meet in LDS at
// the end: rescale to the largest m and add (KW = 4 waves to the 16 rows; at head dimension 256 with many rows one or two, and
// four or two groups of 16 rows to a workgroup).  Eight times as many workgroups as 128-row tiles, chains a quarter as long,
// no workspace, no second launch.  The price: every 16 rows read all keys from the L2 (a 128-row tile shares them), so the
// kernels with larger tiles stay ahead wherever they fill the chip.
//
// All products run on v_mfma_f32_16x16x32_bf16, transposed: S^T = K Q^T, O^T += V^T P~^T, query = MFMA column (lane % 16).
// With kg = lane / 16 a lane holds the scores of keys 4 kg .. + 3 and 16 + 4 kg .. + 3 of its query, which are the B
// operand of a value product over the block's 32 keys as they stand.
//   score step (key tile a, t): A = K[key 16 a + lane % 16][32 t + 8 kg .. + 7], B = Q[query][32 t + 8 kg .. + 7]
//   value tile (cq, e): A = V[the lane's 8 keys][column 16 VW cq + VW (lane % 16) + e], so that a lane reads VW
//   neighbouring columns of a key row at once; MFMA row x of the result is column 16 VW cq + VW x + e
// K and V come straight from global memory into the registers that feed the matrix pipe (no wave shares them), V of the
// block while its scores are formed, K of the next one behind them.  Q and tQ are the same for all waves: in LDS, as the
// MFMAs read them.
//
// fp32 accuracy from bf16 products: an fp32 number from 2^-110 up is EXACTLY the sum of three bf16 numbers (x = hi + mid + lo,
// each the leading 8 bits of what is left), so there is no scale to choose.  Below, lo and then mid fall under bf16's smallest
// subnormal; see SMALL.  fp32 x fp32: the six products down to 2^-24 of the largest (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi).  bf16
// inputs are one term; their weights P~, H~ are split like fp32 ones, three products.  Against the fp32 MFMAs, a sixteenth as
// fast, that is 2.7 and 5.3 to 16 times less matrix time.  Infinities and NaN do not survive the split (inf - inf): a tile with a
// result that is not finite, or that may hang on numbers too small for the split, is redone with fp32 products.
//
// Bound by latency (one or two waves per SIMD, 75 % of their time waiting) and by the loads: 64 KiB per wave and block at d = 256 in
// bf16, twice that in fp32.  Measured, kernel alone, us, before -> now (d <= 128: the tile kernels; d = 256: fp32 MFMAs, 64 rows to
// a workgroup): fp32 B1 H2 L256 d64 26 -> 12.4; bf16 B1 H8 Lq300 Lkv77 d64, no key tangents 8.5 -> 4.5; bf16 B1 H4 L512 d128 29 ->
// 15; fp32 B2 H3 L446 d96 55 -> 29; d = 256, bf16: L3203 1713 -> 142, L2856 without tangents 585 -> 60, B4 H24 L77 58 -> 26; fp32:
// 1729 -> 347, 563 -> 126, 60 -> 46.  Errors against 64 bits (relative 2-norm of o, to, lse): fp32 d64 2.7e-7, 3.3e-7, 3.9e-8 -> 2.3e-7,
// 2.6e-7, 3.3e-8; d = 256 at logit std 8 6.2e-7, 1.3e-6, 4.4e-8 -> 5.0e-7, 8.9e-7, 3.9e-8; bf16 inputs 2.5e-6 (pairs) -> 2.4e-7.
#pragma once
#include "launchers.h"
#include <hip/hip_bf16.h>
#include <type_traits>
#include <utility>
#include <stdint.h>

namespace attn_jvp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int BR = 16, BC = 32;              // query rows of a workgroup, keys of a block
constexpr int TAN_NONE = 0, TAN_QUERY = 1, TAN_ALL = 2;
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;
constexpr float LOG2E_REST = (float)(1.4426950408889634 - (double)LOG2E);
// Nats by which a row's scores may exceed m before m is moved.  The weights are exp(S - (m + MAX_SLACK)), never above 1, so that
// values up to the end of the fp32 range stay in it; the price, weights that flush to zero MAX_SLACK nats earlier, is why
// there are few.
constexpr float MAX_SLACK = 4.f;

// A term that falls away is below 2^-126, whichever number it is of.  A sum or result of at least SMALL does not show it, unless
// a factor above LARGE is behind it: K, tK meet Q, tQ, which are looked at one by one (what is small beside others of its
// sum costs nothing, but that is not known there); V, tV show in o, to (of bf16 inputs, exact as they are, neither) and the tangent
// scores in rowsum(P o tS), so that the keys cost nothing to check.  Not seen: a weight below 2^-102 of its row's sum whose V is
// above 2^78 times the row's result, and values below half of bf16's smallest subnormal, which come out as zero.
// Measured: the check 0 to 2.6 % of a call (fp32 B1 H2 L256 d64 13.6 -> 13.9 us, 8 heads L300 d256 48.5 -> 48.9); a call whose tiles are
// all redone 2.1 to 2.5 times the time in fp32, 2.9 to 3.8 times in bf16.  fp32 V x 1e-36: o 5e-5 out in the 2-norm -> 6e-7, tangents x 1e-36:
// to 3e-3 -> 7e-7.
constexpr float SMALL = 0x1p-80f, LARGE = 0x1p22f;
// What of a tile is redone: o and lse apart from to, so that they have the same bits with and without tangents, whatever those are.
constexpr int REDO_O = 1, REDO_TO = 2, O_NOT_FINITE = 4, TO_NOT_FINITE = 8;
// The factor on V, tV where a result is not finite, so that the sums over up to 2^24 keys of values up to the end of the range stay
// in it: the weights are at most 1 each, not in all.  (What of that tile is below 2^-102 loses bits to the factor.)
constexpr float DOWN = 0x1p-24f;

#define FENCE() __builtin_amdgcn_sched_barrier(0)      // no instruction is scheduled across this point

template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {      // f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
    static_for_impl<N>(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}
__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// x - term, term one half of a packed bf16 pair: one instruction, unpacking included (exact: the result is representable).
// `minus_one` is that constant in the half it takes, from a scalar register: as an inline constant it would land in the other.
__device__ __forceinline__ float less_half(uint32_t pair, uint32_t minus_one, float x) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, minus_one), x, false);
}
__device__ __forceinline__ uint32_t high_halves(float lo, float hi) {      // bf16 truncations of two numbers, packed
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
// N sets of eight fp32 numbers as the packed bf16 terms of their sums.  hi is rounded, so that what is left has either sign and
// the products that are dropped average out; mid is truncated (a byte permutation, half the cost of the conversion), lo is
// exact.  Cut into OPS instructions, stage by stage over all sets: a dot product's result may be read three instructions
// later at the earliest.
template <int N>
struct Split {
    static constexpr int PAIRS = 4 * N, OPS = 7 * PAIRS;
    float x[8 * N], rest[8 * N];
    uint32_t low = 0x0000bf80u, high = 0xbf800000u;
    __device__ __forceinline__ Split() { asm("" : "+s"(low), "+s"(high)); }
    template <int OP>
    __device__ __forceinline__ void op(u32x4 (&term)[N][3]) {
        if constexpr (OP < PAIRS) {
            const f32x2 v = {x[2 * OP], x[2 * OP + 1]};
            term[OP / 4][0][OP % 4] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
        } else if constexpr (OP < 3 * PAIRS) {
            constexpr int i = OP - PAIRS;
            rest[i] = less_half(term[i / 8][0][i / 2 % 4], i & 1 ? high : low, x[i]);
        } else if constexpr (OP < 4 * PAIRS) {
            constexpr int j = OP - 3 * PAIRS;
            term[j / 4][1][j % 4] = high_halves(rest[2 * j], rest[2 * j + 1]);
        } else if constexpr (OP < 6 * PAIRS) {
            constexpr int i = OP - 4 * PAIRS;
            rest[i] = less_half(term[i / 8][1][i / 2 % 4], i & 1 ? high : low, rest[i]);
        } else {
            constexpr int j = OP - 6 * PAIRS;
            term[j / 4][2][j % 4] = high_halves(rest[2 * j], rest[2 * j + 1]);
        }
    }
    __device__ __forceinline__ void all(u32x4 (&term)[N][3]) {
        static_for<OPS>([&](auto I) __attribute__((always_inline)) { op<decltype(I)::value>(term); });
    }
};
// The smallest magnitude of the numbers given, zeros left out.
struct Smallest {
    uint32_t least = ~0u;                                                          // bits without sign, less one
    __device__ __forceinline__ void see(float x) {
        const uint32_t bits = 2 * __float_as_uint(x) - 1;
        least = bits < least ? bits : least;
    }
    __device__ __forceinline__ bool below(float limit) const { return least < 2 * __float_as_uint(limit) - 1; }
};
// maximum and sum over the four lanes that share a query (lane, lane ^ 16, lane ^ 32, lane ^ 48)
__device__ __forceinline__ float row_max(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row_sum(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// e^x, x <= 0: v_exp_f32 is good to an ulp, but x log2(e), rounded, is out by 2^-24 of itself, which is the larger error from
// e^-2 down.  The rounding of the product, and of the constant, come back as a correction of first order.
__device__ __forceinline__ float exp_nat(float x) {
    const float t = x * LOG2E;
    const float r = fmaf(x, LOG2E_REST, fmaf(x, LOG2E, -t));
    const float e = __builtin_amdgcn_exp2f(t);
    return x < -200.f ? 0.f : fmaf(e, r * LN2, e);       // (-inf too, where the correction is NaN)
}

// Eight consecutive elements of a row as loaded, and W neighbouring columns of a key row.
template <typename T> struct In;
template <> struct In<float> {
    static constexpr int TERMS = 3;          // bf16 terms of an element
    static constexpr int MAX_VW = 4;         // columns of a 16-byte load
    struct Row8 { f32x4 a, b; };
    static __device__ __forceinline__ Row8 load8(const float* p) {
        return Row8{*reinterpret_cast<const f32x4*>(p), *reinterpret_cast<const f32x4*>(p + 4)};
    }
    static __device__ __forceinline__ void up(const Row8& r, float (&x)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[i] = r.a[i]; x[4 + i] = r.b[i]; }
    }
    template <int W> struct Cols { typedef float type __attribute__((ext_vector_type(W))); };
    template <int W> static __device__ __forceinline__ typename Cols<W>::type load_cols(const float* p) {
        return *reinterpret_cast<const typename Cols<W>::type*>(p);
    }
    template <int W> static __device__ __forceinline__ float col(typename Cols<W>::type v, int e) { return v[e]; }
};
template <> struct In<__hip_bfloat16> {
    static constexpr int TERMS = 1;
    static constexpr int MAX_VW = 8;
    typedef u32x4 Row8;
    static __device__ __forceinline__ Row8 load8(const __hip_bfloat16* p) { return *reinterpret_cast<const u32x4*>(p); }
    static __device__ __forceinline__ void up(const Row8& r, float (&x)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[2 * i] = __uint_as_float(r[i] << 16); x[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u); }
    }
    template <int W> struct Cols { struct type { uint32_t d[W / 2]; }; };      // W / 2 dwords
    template <int W> static __device__ __forceinline__ typename Cols<W>::type load_cols(const __hip_bfloat16* p) {
        typename Cols<W>::type r;
        if constexpr (W == 8) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(p);
            r.d[0] = v[0]; r.d[1] = v[1]; r.d[2] = v[2]; r.d[3] = v[3];
        } else if constexpr (W == 4) {
            const u32x2 v = *reinterpret_cast<const u32x2*>(p);
            r.d[0] = v[0]; r.d[1] = v[1];
        } else {
            r.d[0] = *reinterpret_cast<const uint32_t*>(p);
        }
        return r;
    }
    template <int W> static __device__ __forceinline__ float col(const typename Cols<W>::type& v, int e) {
        return __uint_as_float(e & 1 ? v.d[e / 2] & 0xffff0000u : v.d[e / 2] << 16);
    }
    // a value operand: the same half of the eight rows' dwords
    template <int W> static __device__ __forceinline__ u32x4 column(const typename Cols<W>::type (&v)[8], int e) {
        u32x4 t;
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = __builtin_amdgcn_perm(v[2 * j + 1].d[e / 2], v[2 * j].d[e / 2], e & 1 ? 0x07060302u : 0x05040100u);
        return t;
    }
};

template <typename TIn, int D, int TAN, int KW, int OCC_ASKED>      // KW: waves that share 16 query rows and deal their keys among them
struct Cfg {
    static constexpr bool TANGENT = TAN != TAN_NONE, KV_TANGENT = TAN == TAN_ALL;
    static constexpr bool BF16 = In<TIn>::TERMS == 1;
    static constexpr int NW = 4, NTHREADS = 64 * NW;
    static constexpr int GROUPS = NW / KW, ROWS = BR * GROUPS;     // of 16 rows to a workgroup; its rows
    // workgroups that share a compute unit, where the registers allow it and there are that many (OCC_ASKED).  Alone on its unit
    // one has 512 registers to a lane: keys, values and operands ahead of their use, nothing spilled (fp32 B1 H8 L512 d64 23.2 -> 20.1
    // us, bf16 B1 H4 L512 d128 17.9 -> 15.3, with the steps beside it).
    static constexpr int OCC = D * sizeof(TIn) <= 256 ? OCC_ASKED : 1;
    static constexpr int NT = D / 32;                              // score steps
    // Columns a lane reads of a key row at once: 16 bytes of them as a rule, as many as divide the row; two where the registers
    // of a wider group would spill (head dimension 256 with tangents: fp32 426 -> 348 us, bf16 158 -> 141 at 3203 keys).
    static constexpr int VW = D == 256 && (TAN == TAN_ALL || (BF16 && TANGENT)) ? 2
                              : D % (16 * In<TIn>::MAX_VW) == 0 ? In<TIn>::MAX_VW : D % 64 == 0 ? 4 : 2;
    static constexpr int NCQ = D / (16 * VW);                      // column groups; a group is VW value tiles
    // What is requested ahead.  Keys: the next block's behind the scores; where a whole block does not fit beside the
    // accumulators (ROLL) a ring of K_RING score steps, each requested again once it is split.  Column groups of V: all
    // before the scores, or one before the block's second score tile and each one a group ahead.
    static constexpr bool ROLL = D * sizeof(TIn) >= 1024 || (D * sizeof(TIn) >= 512 && (!BF16 || TANGENT)) ||
                                 (OCC == 2 && D * sizeof(TIn) >= 256 && KV_TANGENT);      // (a spilled prefetch waits for memory: bf16 d256 H8 Lq2000 Lkv300 62.6 -> 48.7 us)
    static constexpr int K_RING = !ROLL ? 2 * NT : NT >= 8 ? NT / 2 : NT;
    static constexpr int V_GROUP_REGS = (KV_TANGENT ? 2 : 1) * 8 * VW * (int)sizeof(TIn) / 4;
    static constexpr int V_AHEAD = NCQ * V_GROUP_REGS <= (D == 256 ? 64 : 128) ? NCQ : 1;
    // ... the first block's beside its keys and the next one's behind a block's products, where there is room, else when a block begins
    static constexpr bool V_EARLY = V_AHEAD == NCQ && OCC == 1 && D * sizeof(TIn) <= 256;
    static constexpr int V_SLOTS = V_AHEAD < NCQ ? V_AHEAD + 1 : V_AHEAD;
    // Operands from Q and tQ are read from LDS a score step ahead where the registers allow.
    static constexpr bool Q_AHEAD = OCC == 1 && !(D == 256 && KV_TANGENT);
    static constexpr int Q_PLANE = NT * 1024;                      // bytes: [step][lane] 16-byte operands
    static constexpr int Q_BYTES = (TANGENT ? 2 : 1) * In<TIn>::TERMS * Q_PLANE;      // of a group
    static constexpr int OUT_ROW = D + 4;                          // floats; 4 of padding spread the rows over the banks
    static constexpr int PART_BYTES = (TANGENT ? 2 : 1) * BR * OUT_ROW * 4;       // a wave's O~, A + B
    static constexpr int STATE_BASE = NW * PART_BYTES > GROUPS * Q_BYTES ? NW * PART_BYTES : GROUPS * Q_BYTES;
    static constexpr int LDS_BYTES = STATE_BASE + NW * BR * 16;    // + m, l, r, row maximum of each wave and row
    static_assert(LDS_BYTES * OCC <= 160 * 1024, "fits a compute unit");
};

template <typename TIn, int D, int TAN, int KW, int OCC_ASKED, bool FAR>      // FAR: 64-bit row offsets (rows_far_apart)
__global__ __launch_bounds__((Cfg<TIn, D, TAN, KW, OCC_ASKED>::NTHREADS), (Cfg<TIn, D, TAN, KW, OCC_ASKED>::OCC)) void attn_jvp_keysplit_kernel(
    const TIn* __restrict__ Q, const TIn* __restrict__ K, const TIn* __restrict__ V,
    const TIn* __restrict__ tQ, const TIn* __restrict__ tK, const TIn* __restrict__ tV,
    void* __restrict__ O, void* __restrict__ tO, float* __restrict__ LSE,
    int Lq, int Lkv, float scale, int q_tiles, int H, int blhd, int out_bf16) {
    // (the instantiations must agree bit for bit, absent tangents against zero ones: no implicit fusing)
#pragma clang fp contract(off)
    using C = Cfg<TIn, D, TAN, KW, OCC_ASKED>;
    using I = In<TIn>;
    using Row8 = typename I::Row8;
    using Cols = typename I::template Cols<C::VW>::type;
    constexpr bool TANGENT = C::TANGENT, KV_TANGENT = C::KV_TANGENT;
    constexpr int NT = C::NT, VW = C::VW, NCQ = C::NCQ, TERMS = I::TERMS, NTILES = D / 16;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    // (all arguments are asked for at once: one wait for memory at the start, not one in front of each use)
    asm volatile("" :: "s"(Q), "s"(K), "s"(V), "s"(tQ), "s"(tK), "s"(tV), "s"(Lq), "s"(Lkv), "s"(q_tiles), "s"(H), "s"(blhd));

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, kg = lane >> 4;
    const int kw = wave % KW, group = wave / KW;       // the wave's share of the keys, and its rows
    // workgroups go round-robin over the 8 XCDs: a contiguous range of tiles for each, so that they share their keys in L2
    const int n_wg = gridDim.x;
    const int bid = (n_wg & 7) == 0 ? (int)(blockIdx.x & 7) * (n_wg >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const long bh = (int)((unsigned)bid / (unsigned)q_tiles);
    const int q0 = (bid % q_tiles) * C::ROWS;
    // [B,H,L,d]: rows of a head contiguous; [B,L,H,d]: rows of a head H*d elements apart
    const long row_elems = blhd ? (long)H * D : D;
    long q_base = bh * (long)Lq * D, kv_base = bh * (long)Lkv * D;
    if (blhd) {
        const long bidx = bh / H, hidx = bh % H;
        q_base = (bidx * Lq * H + hidx) * D;
        kv_base = (bidx * Lkv * H + hidx) * D;
    }
    const int n_blocks = (Lkv + BC - 1) / BC;

    // ---- loads (rows past the end repeat the last key: their weights are zero) ----
    // A row is a uniform address, its block's first row, plus 32 bits that are the lane's own and stay as they are from block to
    // block, up to a ragged last one: per block and row a 64-bit product of row number and stride took 0.3 us of 3.5.  (32 rows are
    // below 4 GiB: checked on the host, which takes FAR where they are not.)
    using Off = std::conditional_t<FAR, uint64_t, uint32_t>;
    const long row_bytes = row_elems * (long)sizeof(TIn);
    const Off row_step = (Off)row_bytes;
    auto my_key = [&](int i) __attribute__((always_inline)) { return 16 * (i >> 2) + 4 * kg + (i & 3); };      // of the block: the lane's i-th
    auto live_of = [&](int blk) __attribute__((always_inline)) { const int left = Lkv - blk * BC; return left < BC ? left : BC; };      // keys of a block that exist
    auto block_at = [&](const TIn* X, int blk) __attribute__((always_inline)) {
        return reinterpret_cast<const char*>(X) + kv_base * (long)sizeof(TIn) + (long)blk * BC * row_bytes;
    };
    Off k_off[2], v_off[8];
    auto set_k_rows = [&](int a, int live) __attribute__((always_inline)) {
        const int row = 16 * a + c;
        k_off[a] = (Off)(row < live ? row : live - 1) * row_step + 8 * kg * (uint32_t)sizeof(TIn);
    };
    auto set_v_rows = [&](int live) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v_off[i] = (Off)(my_key(i) < live ? my_key(i) : live - 1) * row_step + VW * c * (uint32_t)sizeof(TIn);
    };
    Row8 kr[C::K_RING], tkr[KV_TANGENT ? C::K_RING : 1];
    Cols vr[C::V_SLOTS][8], tvr[KV_TANGENT ? C::V_SLOTS : 1][8];
    auto load_k_step = [&](int step, int blk) __attribute__((always_inline)) {      // step NT a + t of a block: key tile a, score step t
        const Off at = k_off[step / NT];
        kr[step % C::K_RING] = I::load8(reinterpret_cast<const TIn*>(block_at(K, blk) + at) + 32 * (step % NT));
        if constexpr (KV_TANGENT) tkr[step % C::K_RING] = I::load8(reinterpret_cast<const TIn*>(block_at(tK, blk) + at) + 32 * (step % NT));
    };
    // Past the last block (behind a wave's last, and for waves without any) requests are for nothing: of one row that is there, for all
    // lanes.  As the last block's rows again they took the way to the L2 that V is waiting for: fp32 d = 256 without tangents, H32 Lq503
    // Lkv27 22.9 us a call, now 21.3 (31 x 656 x 27 41.3 -> 38.8).
    auto next_block = [&](int blk, int* live) __attribute__((always_inline)) {
        *live = blk < n_blocks ? live_of(blk) : 1;
        return blk < n_blocks ? blk : n_blocks - 1;
    };
    auto k_tile = [&](int a, int blk) __attribute__((always_inline)) {      // tile a of a block is next
        int live;
        const int b = next_block(blk, &live);
        if (live < BC) set_k_rows(a, live);
        return b;
    };
    auto load_k = [&](int blk) __attribute__((always_inline)) {      // as much of a block as the ring holds
#pragma unroll
        for (int a = 0; a * NT < C::K_RING; ++a) {
            const int b = k_tile(a, blk);
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (NT * a + t < C::K_RING) load_k_step(NT * a + t, b);
        }
    };
    auto load_v = [&](auto G, int blk) __attribute__((always_inline)) {
        constexpr int cq = decltype(G)::value, slot = cq % C::V_SLOTS;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            vr[slot][i] = I::template load_cols<VW>(reinterpret_cast<const TIn*>(block_at(V, blk) + v_off[i]) + 16 * VW * cq);
            if constexpr (KV_TANGENT) tvr[slot][i] = I::template load_cols<VW>(reinterpret_cast<const TIn*>(block_at(tV, blk) + v_off[i]) + 16 * VW * cq);
        }
    };
    auto load_first_v = [&](int blk) __attribute__((always_inline)) {
        int live;
        const int b = next_block(blk, &live);
        if (live < BC) set_v_rows(live);
        static_for<C::V_AHEAD>([&](auto G) { load_v(G, b); });
    };
    using A0 = std::integral_constant<int, 0>;
    using A1 = std::integral_constant<int, 1>;
    // ---- Q, tQ into LDS as B operands: lane l of step t holds row l % 16, elements 32 t + 8 (l / 16) .. + 7 ----
    // Requested first, where a lane has few of them: loads return in order, so that Q is split while the first block's keys and
    // values are under way (fp32 B1 H2 L256 d64: 2.9 us from the start to the scores behind the keys).
    constexpr int Q_ITEMS = C::GROUPS * (TANGENT ? 2 : 1) * NT * 64, Q_PER_LANE = (Q_ITEMS + C::NTHREADS - 1) / C::NTHREADS;
    constexpr bool Q_FIRST = Q_PER_LANE <= 4;
    int redo = 0;                            // with fp32 products: REDO_*
    auto q_load = [&](int idx) __attribute__((always_inline)) -> Row8 {
        const int at_group = idx / ((TANGENT ? 2 : 1) * NT * 64), which = idx / (NT * 64) % (TANGENT ? 2 : 1), t = idx / 64 % NT, l = idx & 63;
        const int wanted = q0 + BR * at_group + (l & 15), row = wanted < Lq ? wanted : Lq - 1;       // rows past the end repeat the last one and are not stored
        return I::load8((which ? tQ : Q) + q_base + (long)row * row_elems + 32 * t + 8 * (l >> 4));
    };
    auto q_store = [&](int idx, const Row8& r) __attribute__((always_inline)) {
        const int at_group = idx / ((TANGENT ? 2 : 1) * NT * 64), which = idx / (NT * 64) % (TANGENT ? 2 : 1), t = idx / 64 % NT, l = idx & 63;
        char* at = smem + at_group * C::Q_BYTES + which * TERMS * C::Q_PLANE + t * 1024 + l * 16;
        if constexpr (TERMS == 3) {
            Split<1> split;
            u32x4 term[1][3];
            float x[8];
            I::up(r, x);
            Smallest small;
            float top = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                split.x[i] = x[i];
                small.see(x[i]);
                top = fmaxf(top, fabsf(x[i]));
            }
            if (__builtin_amdgcn_ballot_w64(small.below(SMALL) || top > LARGE) != 0) redo |= which ? REDO_TO : REDO_O | REDO_TO;      // (`which` is the wave's)
            split.all(term);
#pragma unroll
            for (int y = 0; y < 3; ++y) *reinterpret_cast<u32x4*>(at + y * C::Q_PLANE) = term[0][y];
        } else {
            *reinterpret_cast<u32x4*>(at) = __builtin_bit_cast(u32x4, r);
        }
    };
    Row8 q_raw[Q_FIRST ? Q_PER_LANE : 1];
    if constexpr (Q_FIRST) {
#pragma unroll
        for (int n = 0; n < Q_PER_LANE; ++n) {
            const int idx = tid + C::NTHREADS * n;
            if (Q_ITEMS % C::NTHREADS == 0 || idx < Q_ITEMS) q_raw[n] = q_load(idx);
        }
        FENCE();
    }
    set_k_rows(0, BC);
    set_k_rows(1, BC);
    set_v_rows(BC);
    // (by waves without a block too: behind a branch the compiler would wait for everything before Q is split)
    load_k(kw);
    if constexpr (C::V_EARLY) load_first_v(kw);
    FENCE();
    if constexpr (Q_FIRST) {
#pragma unroll
        for (int n = 0; n < Q_PER_LANE; ++n) {
            const int idx = tid + C::NTHREADS * n;
            if (Q_ITEMS % C::NTHREADS == 0 || idx < Q_ITEMS) q_store(idx, q_raw[n]);
        }
    } else {
        for (int idx = tid; idx < Q_ITEMS; idx += C::NTHREADS) q_store(idx, q_load(idx));
    }
    redo = __builtin_amdgcn_readfirstlane(redo);
    __syncthreads();
    auto q_term = [&](int which, int x, int t) __attribute__((always_inline)) {
        return *reinterpret_cast<const u32x4*>(smem + group * C::Q_BYTES + (which * TERMS + x) * C::Q_PLANE + t * 1024 + lane * 16);
    };

    f32x4 acc_o[NTILES], acc_t[TANGENT ? NTILES : 1];      // [VW cq + e][r]: column 16 VW cq + VW (4 kg + r) + e of query c
    float m, row_top, l, r_sum;                            // l, r: this lane's keys only until the sweep's end
    auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NTILES; ++n) {
            acc_o[n] = f32x4{};
            if constexpr (TANGENT) acc_t[n] = f32x4{};
        }
        m = -INFINITY; row_top = -INFINITY; l = 0.f; r_sum = 0.f;
    };
    // Scores of the lane's eight keys -> weights p, h; the reference m trails the row maximum by up to MAX_SLACK.  Straight-line code
    // over the eight, with the keys past the end set aside in the one block that has any: a branch around each weight, which is
    // what a choice between zero and an exponential compiles to, made a chain of eight (0.5 us per block).
    auto weights = [&](int blk, float (&s)[8], float (&ts)[8], float (&p)[8], float (&h)[8]) __attribute__((always_inline)) {
        const int live = live_of(blk);
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = s[i] * scale;
        if (live < BC)                               // (uniform)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (my_key(i) >= live) { x[i] = -INFINITY; ts[i] = 0.f; }
        float mb = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
        mb = row_max(mb);
        row_top = fmaxf(row_top, mb);                // the maximum itself, for lse: m + log l would round twice as often
        const float m_new = mb > m + MAX_SLACK ? mb : m;
        float alpha = 1.f;
        if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {
            const float back = exp_nat(m - m_new);
            alpha = m_new == m ? 1.f : back;         // 0 when the first finite score comes (m = -inf)
#pragma unroll
            for (int n = 0; n < NTILES; ++n) {
                acc_o[n] *= alpha;
                if constexpr (TANGENT) acc_t[n] *= alpha;
            }
        }
        m = m_new;
        const float m_ref = m == -INFINITY ? 0.f : m + MAX_SLACK;       // (scores of -inf so far: weight 0, not NaN)
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = fmaf(s[i], scale, -m_ref);
        if (live < BC)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (my_key(i) >= live) x[i] = -INFINITY;
        float row_p = 0.f, row_h = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            p[i] = exp_nat(x[i]);
            row_p += p[i];
            h[i] = TANGENT ? p[i] * (ts[i] * scale) : 0.f;
            row_h += h[i];
        }
        l = fmaf(alpha, l, row_p);
        r_sum = fmaf(alpha, r_sum, row_h);
    };

    // ---- the sweep on split products ----
    // Six products of terms (X, Y) for three-term operands, the large one first or last; of a step's or tile's products those
    // that share a sum do not follow each other.  The instructions that split the next step's operands go behind them, three
    // to each: a product takes the matrix pipe 16 cycles, its issue and theirs 4 each.
    constexpr int PRODUCTS = KV_TANGENT ? 3 : TANGENT ? 2 : 1;
    constexpr int X[6] = {0, 0, 2, 1, 0, 1}, Y[6] = {0, 2, 0, 1, 1, 0};
    constexpr int SETS = KV_TANGENT ? 2 : 1;
    auto score_tile = [&](auto A, int blk, float (&s)[8], float (&ts)[8]) __attribute__((always_inline)) {
        constexpr int a = decltype(A)::value;
        // ring: the block of the step K_RING ahead, in this tile or the next (behind the wave's last block: for nothing)
        int next = blk;
        if constexpr (C::ROLL) next = a == 0 ? k_tile(1, blk) : k_tile(0, blk + KW);
        // the large products on a sum of their own for every two steps (a chain of eight steps would carry twice the rounding
        // error), and the small ones on one
        constexpr int NS = (NT + 1) / 2;
        f32x4 hi[NS], thi[NS], lo = {}, tlo = {};
#pragma unroll
        for (int i = 0; i < NS; ++i) { hi[i] = f32x4{}; thi[i] = f32x4{}; }
        auto request = [&](int t) __attribute__((always_inline)) {       // step t has been taken: its ring slot's next content
            const int step = NT * a + t;
            if constexpr (C::ROLL) load_k_step((step + C::K_RING) % (2 * NT), t + C::K_RING >= NT ? next : blk);
        };
        if constexpr (TERMS == 3) {
            Split<SETS> split;
            u32x4 term[2][SETS][3], q[2][3], tq[2][3];
            auto read_q = [&](int t) __attribute__((always_inline)) {
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    q[t % 2][x] = q_term(0, x, t);
                    if constexpr (TANGENT) tq[t % 2][x] = q_term(1, x, t);
                }
            };
            auto take = [&](int t) __attribute__((always_inline)) {
                const int slot = (NT * a + t) % C::K_RING;
                float x[8];
                I::up(kr[slot], x);
#pragma unroll
                for (int i = 0; i < 8; ++i) split.x[i] = x[i];
                if constexpr (KV_TANGENT) {
                    I::up(tkr[slot], x);
#pragma unroll
                    for (int i = 0; i < 8; ++i) split.x[(SETS - 1) * 8 + i] = x[i];
                }
            };
            if constexpr (C::Q_AHEAD) read_q(0);
            take(0);
            split.all(term[0]);
            request(0);
            static_for<NT>([&](auto T) __attribute__((always_inline)) {
                constexpr int t = decltype(T)::value;
                if constexpr (!C::Q_AHEAD) read_q(t);
                else if constexpr (t + 1 < NT) read_q(t + 1);
                if constexpr (t + 1 < NT) take(t + 1);
                static_for<6 * PRODUCTS>([&](auto J) __attribute__((always_inline)) {
                    constexpr int j = decltype(J)::value, i = j / PRODUCTS, which = PRODUCTS == 1 ? 0 : (j % PRODUCTS + 1) % 2 + (j % PRODUCTS == 2 ? 1 : 0);
                    f32x4& sum = i == 0 ? (which == 0 ? hi[t / 2] : thi[t / 2]) : which == 0 ? lo : tlo;
                    if constexpr (which == 0) sum = mfma(term[t & 1][0][X[i]], q[t & 1][Y[i]], sum);
                    else if constexpr (which == 1) sum = mfma(term[t & 1][0][X[i]], tq[t & 1][Y[i]], sum);
                    else sum = mfma(term[t & 1][SETS - 1][X[i]], q[t & 1][Y[i]], sum);
                    if constexpr (t + 1 < NT)
                        static_for<Split<SETS>::OPS>([&](auto U) __attribute__((always_inline)) {
                            constexpr int u = decltype(U)::value;
                            if constexpr (u * 6 * PRODUCTS / Split<SETS>::OPS == j) split.template op<u>(term[(t + 1) & 1]);
                        });
                    FENCE();
                });
                if constexpr (t + 1 < NT) request(t + 1);
            });
        } else {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int slot = (NT * a + t) % C::K_RING;
                const u32x4 k = __builtin_bit_cast(u32x4, kr[slot]), q = q_term(0, 0, t);
                hi[t / 2] = mfma(k, q, hi[t / 2]);
                if constexpr (TANGENT) thi[t / 2] = mfma(k, q_term(1, 0, t), thi[t / 2]);
                if constexpr (KV_TANGENT) thi[t / 2] = mfma(__builtin_bit_cast(u32x4, tkr[slot]), q, thi[t / 2]);
                request(t);
                if constexpr (C::ROLL) FENCE();
            }
        }
        auto total = [](f32x4 (&x)[NS]) __attribute__((always_inline)) {
            if constexpr (NS == 4) return (x[0] + x[1]) + (x[2] + x[3]);
            else if constexpr (NS == 2) return x[0] + x[1];
            else return x[0];
        };
        if constexpr (TERMS == 3) { hi[0] += lo; thi[0] += tlo; }
        const f32x4 su = total(hi), tu = total(thi);
#pragma unroll
        for (int i = 0; i < 4; ++i) { s[4 * a + i] = su[i]; ts[4 * a + i] = tu[i]; }
    };
    auto values = [&](int blk, const u32x4 (&p)[3], const u32x4 (&h)[3]) __attribute__((always_inline)) {
        auto next_group = [&](auto G) __attribute__((always_inline)) {
            constexpr int cq = decltype(G)::value;
            if constexpr (cq + C::V_AHEAD < NCQ) {
                load_v(std::integral_constant<int, cq + C::V_AHEAD>{}, blk);
                FENCE();
            }
        };
        if constexpr (TERMS == 3) {
            Split<SETS> split;
            u32x4 term[2][SETS][3];
            auto take = [&](auto Nc) __attribute__((always_inline)) {
                constexpr int n = decltype(Nc)::value, slot = n / VW % C::V_SLOTS;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    split.x[i] = I::template col<VW>(vr[slot][i], n % VW);
                    if constexpr (KV_TANGENT) split.x[(SETS - 1) * 8 + i] = I::template col<VW>(tvr[slot][i], n % VW);
                }
            };
            take(std::integral_constant<int, 0>{});
            split.all(term[0]);
            static_for<NTILES>([&](auto Nc) __attribute__((always_inline)) {
                constexpr int n = decltype(Nc)::value;
                if constexpr (n % VW == 0) next_group(std::integral_constant<int, n / VW>{});
                if constexpr (n + 1 < NTILES) take(std::integral_constant<int, n + 1>{});
                static_for<6 * PRODUCTS>([&](auto J) __attribute__((always_inline)) {
                    constexpr int j = decltype(J)::value, i = 5 - j / PRODUCTS, which = PRODUCTS == 1 ? 0 : (j % PRODUCTS + 1) % 2 + (j % PRODUCTS == 2 ? 1 : 0);
                    if constexpr (which == 0) acc_o[n] = mfma(term[n & 1][0][X[i]], p[Y[i]], acc_o[n]);
                    else if constexpr (which == 1) acc_t[n] = mfma(term[n & 1][0][X[i]], h[Y[i]], acc_t[n]);
                    else acc_t[n] = mfma(term[n & 1][SETS - 1][X[i]], p[Y[i]], acc_t[n]);
                    if constexpr (n + 1 < NTILES)
                        static_for<Split<SETS>::OPS>([&](auto U) __attribute__((always_inline)) {
                            constexpr int u = decltype(U)::value;
                            if constexpr (u * 6 * PRODUCTS / Split<SETS>::OPS == j) split.template op<u>(term[(n + 1) & 1]);
                        });
                    FENCE();
                });
            });
        } else {
            static_for<NTILES>([&](auto Nc) __attribute__((always_inline)) {
                constexpr int n = decltype(Nc)::value, slot = n / VW % C::V_SLOTS;
                if constexpr (n % VW == 0) next_group(std::integral_constant<int, n / VW>{});
                const u32x4 v = I::template column<VW>(vr[slot], n % VW);
                u32x4 tv = v;
                if constexpr (KV_TANGENT) tv = I::template column<VW>(tvr[slot], n % VW);
#pragma unroll
                for (int i = 2; i >= 0; --i) {
                    if constexpr (TANGENT) acc_t[n] = mfma(v, h[i], acc_t[n]);
                    acc_o[n] = mfma(v, p[i], acc_o[n]);
                    if constexpr (KV_TANGENT) acc_t[n] = mfma(tv, p[i], acc_t[n]);
                }
                if constexpr (C::ROLL) FENCE();
            });
        }
    };
    auto sweep = [&]() __attribute__((always_inline)) {
        for (int blk = kw; blk < n_blocks; blk += KW) {
            float s[8], ts[8], p[8], h[8];
            if constexpr (C::V_AHEAD == NCQ && !C::V_EARLY) load_first_v(blk);
            FENCE();
            score_tile(A0{}, blk, s, ts);
            if constexpr (C::V_AHEAD < NCQ) {
                FENCE();
                load_first_v(blk);
                FENCE();
            }
            score_tile(A1{}, blk, s, ts);
            FENCE();
            if constexpr (!C::ROLL) {
                if (blk + KW < n_blocks) load_k(blk + KW);
                FENCE();
            }
            weights(blk, s, ts, p, h);
            Split<TANGENT ? 2 : 1> split;
            u32x4 w[TANGENT ? 2 : 1][3];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                split.x[i] = p[i];
                if constexpr (TANGENT) split.x[8 + i] = h[i];
            }
            split.all(w);
            values(blk, w[0], w[TANGENT ? 1 : 0]);
            if constexpr (C::V_EARLY) {
                FENCE();
                if (blk + KW < n_blocks) load_first_v(blk + KW);
            }
        }
    };
    // ---- ... and on fp32 products, for tiles with infinities or NaN: nothing fetched ahead ----
    auto sweep_f32 = [&](float factor) __attribute__((always_inline)) {
        auto key_row = [&](int j) __attribute__((always_inline)) -> long { return kv_base + (long)(j < Lkv ? j : Lkv - 1) * row_elems; };
        const int row = q0 + BR * group + c < Lq ? q0 + BR * group + c : Lq - 1;
        const long qat = q_base + (long)row * row_elems + 8 * kg;
        for (int blk = kw; blk < n_blocks; blk += KW) {
            float s[8], ts[8], p[8], h[8];
#pragma unroll 1
            for (int a = 0; a < 2; ++a) {
                f32x4 su = {}, tu = {};
                const long kat = key_row(blk * BC + 16 * a + c) + 8 * kg;
#pragma unroll 1
                for (int t = 0; t < NT; ++t) {
                    float k[8], tk[8], q[8], tq[8];
                    I::up(I::load8(K + kat + 32 * t), k);
                    I::up(I::load8(Q + qat + 32 * t), q);
                    if constexpr (TANGENT) I::up(I::load8(tQ + qat + 32 * t), tq);
                    if constexpr (KV_TANGENT) I::up(I::load8(tK + kat + 32 * t), tk);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        su = mfma_f32(k[e], q[e], su);
                        if constexpr (TANGENT) tu = mfma_f32(k[e], tq[e], tu);
                        if constexpr (KV_TANGENT) tu = mfma_f32(tk[e], q[e], tu);
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (a == 0) { s[i] = su[i]; ts[i] = tu[i]; }
                    else { s[4 + i] = su[i]; ts[4 + i] = tu[i]; }
            }
            weights(blk, s, ts, p, h);
            static_for<NCQ>([&](auto G) {
                constexpr int cq = decltype(G)::value, slot = cq % C::V_SLOTS;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const long at = key_row(blk * BC + my_key(i)) + 16 * VW * cq + VW * c;
                    vr[slot][i] = I::template load_cols<VW>(V + at);
                    if constexpr (KV_TANGENT) tvr[slot][i] = I::template load_cols<VW>(tV + at);
                }
#pragma unroll
                for (int e = 0; e < VW; ++e)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float v = I::template col<VW>(vr[slot][i], e) * factor;
                        acc_o[VW * cq + e] = mfma_f32(v, p[i], acc_o[VW * cq + e]);
                        if constexpr (TANGENT) acc_t[VW * cq + e] = mfma_f32(v, h[i], acc_t[VW * cq + e]);
                        if constexpr (KV_TANGENT) acc_t[VW * cq + e] = mfma_f32(I::template col<VW>(tvr[slot][i], e) * factor, p[i], acc_t[VW * cq + e]);
                    }
            });
        }
    };

    // ---- the waves' partial states meet in LDS; returns what is not finite or small ----
    auto finish = [&](bool primal, float up) __attribute__((always_inline)) -> int {
        l = row_sum(l);
        r_sum = row_sum(r_sum);
        __syncthreads();                             // everyone is done with Q, tQ (or with the previous states)
        float* part = reinterpret_cast<float*>(smem + wave * C::PART_BYTES) + c * C::OUT_ROW;
#pragma unroll
        for (int cq = 0; cq < NCQ; ++cq)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* at = part + 16 * VW * cq + VW * (4 * kg + r);
#pragma unroll
                for (int e = 0; e < VW; e += 2) {
                    *reinterpret_cast<f32x2*>(at + e) = f32x2{acc_o[VW * cq + e][r], acc_o[VW * cq + e + 1][r]};
                    if constexpr (TANGENT) *reinterpret_cast<f32x2*>(at + BR * C::OUT_ROW + e) = f32x2{acc_t[VW * cq + e][r], acc_t[VW * cq + e + 1][r]};
                }
            }
        f32x4* state = reinterpret_cast<f32x4*>(smem + C::STATE_BASE);
        if (kg == 0) state[wave * BR + c] = f32x4{m, l, r_sum, row_top};
        __syncthreads();
        int odd = 0;
        for (int idx = tid; idx < C::ROWS * (D / 4); idx += C::NTHREADS) {
            const int row = idx / (D / 4), col = 4 * (idx % (D / 4));
            const int part0 = row / BR * KW, part_row = row % BR;        // its group's first wave
            float top = -INFINITY, m_all = -INFINITY, l_row = 0.f, r_row = 0.f;
#pragma unroll
            for (int w = 0; w < KW; ++w) {
                m_all = fmaxf(m_all, state[(part0 + w) * BR + part_row][0]);
                top = fmaxf(top, state[(part0 + w) * BR + part_row][3]);
            }
            f32x4 o = {}, t = {};
#pragma unroll
            for (int w = 0; w < KW; ++w) {
                const f32x4 st = state[(part0 + w) * BR + part_row];
                const float f = st[0] == m_all ? 1.f : exp_nat(st[0] - m_all);
                l_row = fmaf(f, st[1], l_row);
                r_row = fmaf(f, st[2], r_row);
                const float* at = reinterpret_cast<const float*>(smem + (part0 + w) * C::PART_BYTES) + part_row * C::OUT_ROW + col;
                const f32x4 po = *reinterpret_cast<const f32x4*>(at);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = fmaf(f, po[e], o[e]);
                if constexpr (TANGENT) {
                    const f32x4 pt = *reinterpret_cast<const f32x4*>(at + BR * C::OUT_ROW);
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] = fmaf(f, pt[e], t[e]);
                }
            }
            // epilogue (Alg. 2, last lines)
            const float inv_l = 1.f / l_row;
            const float mu = r_row * inv_l;          // rowsum(P o tS)
            const float scaled = inv_l * up;
            float probe = 0.f, probe_t = 0.f;        // NaN once anything is inf or NaN
            Smallest small, small_t;
            if constexpr (TANGENT) small_t.see(mu);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (TANGENT) t[e] = fmaf(-mu, o[e], t[e]) * scaled;
                o[e] *= scaled;
                probe = fmaf(o[e], 0.f, probe);
                if constexpr (TANGENT) probe_t = fmaf(t[e], 0.f, probe_t);
                if constexpr (TERMS == 3) {
                    small.see(o[e]);
                    if constexpr (TANGENT) small_t.see(t[e]);
                }
            }
            if (probe != probe) odd |= O_NOT_FINITE;
            if (probe_t != probe_t) odd |= TO_NOT_FINITE;
            if (small.below(SMALL)) odd |= REDO_O | REDO_TO;
            if (small_t.below(SMALL)) odd |= REDO_TO;
            if (q0 + row < Lq) {
                const long at = q_base + (long)(q0 + row) * row_elems + col;
                if (out_bf16) {                      // (uniform)
                    auto store = [&](void* out, f32x4 x) __attribute__((always_inline)) {
                        alignas(8) __hip_bfloat16 b[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) b[e] = __float2bfloat16(x[e]);
                        *reinterpret_cast<uint2*>(static_cast<__hip_bfloat16*>(out) + at) = *reinterpret_cast<const uint2*>(b);
                    };
                    if (primal) store(O, o);
                    if constexpr (TANGENT) store(tO, t);
                } else {
                    if (primal) *reinterpret_cast<f32x4*>(static_cast<float*>(O) + at) = o;
                    if constexpr (TANGENT) *reinterpret_cast<f32x4*>(static_cast<float*>(tO) + at) = t;
                }
                if (primal && col == 0) {
                    // the hardware's logarithm comes out low by up to half an ulp of its base-2 value: one Newton step
                    const float sum = l_row * expf(m_all + MAX_SLACK - top), y = logf(sum), y_rest = fmaf(sum, expf(-y), -1.f);
                    const float z = top + y, z_rest = fabsf(top) > fabsf(y) ? y - (z - top) : top - (z - y);
                    LSE[(long)bh * Lq + q0 + row] = l_row == 0.f ? -INFINITY : z + (z_rest + y_rest);      // (0: every score is -inf)
                }
            }
        }
        return odd;
    };

    reset();
    sweep();
    redo |= finish(true, 1.f);
    if (__builtin_expect(__syncthreads_or(redo), 0)) {
        auto any = [&](int what) __attribute__((always_inline)) -> bool {
            __syncthreads();                         // everyone has the answer before the next question
            return __syncthreads_or(redo & what);
        };
        const bool o_down = any(O_NOT_FINITE), to_down = any(O_NOT_FINITE | TO_NOT_FINITE), o_again = any(REDO_O | O_NOT_FINITE);
        const bool to_again = TANGENT && !(o_again && o_down == to_down);      // (if nothing of o is flagged, something of to is)
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {       // o, lse and to; to alone
            if (!(pass == 0 ? o_again : to_again)) continue;
            const bool down = pass == 0 ? o_down : to_down;
            reset();
            sweep_f32(down ? DOWN : 1.f);
            finish(pass == 0, down ? 1.f / DOWN : 1.f);
        }
    }
}

template <typename TIn, int D, int TAN, int KW, int OCC_ASKED = 2, bool FAR = false>
hipError_t launch_waves(const Problem& p) {
    using C = Cfg<TIn, D, TAN, KW, OCC_ASKED>;
    const int q_tiles = (p.Lq - 1) / C::ROWS + 1;
    const long long blocks = (long long)q_tiles * p.B * p.H;
    // (never: head dimension 256, which has no other kernel, and fp32 calls that no tile kernel takes are admitted up to 65535 heads,
    // fp32_vector_supports; others come up to keysplit_groups_per_unit, or by launch_keysplit_far)
    if (blocks > 0x7fffffffLL || (!FAR && (p.layout ? (long long)p.H : 1) * p.d * (long long)sizeof(TIn) * BC + p.d * (long long)sizeof(TIn) > 0xffffffffLL)) return hipErrorInvalidValue;
    auto kern = attn_jvp_keysplit_kernel<TIn, D, TAN, KW, OCC_ASKED, FAR>;
    int dev = 0, cus = 0;
    hipError_t e = device_cus(&dev, &cus);
    if constexpr (C::OCC == 2 && OCC_ASKED == 2 && !FAR)
        if (e == hipSuccess && blocks <= cus) return launch_waves<TIn, D, TAN, KW, 1>(p);
    if (e == hipSuccess) e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), C::LDS_BYTES, dev);
    if (e != hipSuccess) return e;
    MainKernelTimer timer(p);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(C::NTHREADS), C::LDS_BYTES, p.stream,
                       (const TIn*)p.q, (const TIn*)p.k, (const TIn*)p.v, (const TIn*)p.tq, (const TIn*)p.tk, (const TIn*)p.tv,
                       p.o, p.to, p.lse, p.Lq, p.Lkv, p.scale, q_tiles, p.H, p.layout, std::is_same<TIn, float>::value ? 0 : p.out_dtype);
    return timer.finish(hipGetLastError());
}

template <typename TIn, int D, int TAN>
hipError_t launch_one(const Problem& p) {
    if constexpr (D == 256) {
        // One wave (fp32 with tangents: two, Q and tQ of four groups do not fit the LDS) to 16 rows, so that no wave is without a
        // block where there are fewer than four, and fewer partial states meet.  Rounds of workgroups over the units times a round's
        // length in key blocks: a workgroup's fixed part is worth 1.2 blocks, 1.6 with two groups, 4 with four.  Measured, us, four
        // waves to 16 rows -> this: bf16, no key tangents, H16 Lq26057 Lkv25 1154 -> 719, H8 Lq4000 Lkv60 93 -> 55, Lq2000 Lkv300
        // 81 -> 64; fp32 H24 Lq2632 Lkv47 234 -> 154, all tangents H24 L300 96 -> 80.  Where it stays with four, one would
        // take H4 Lq2000 Lkv120 27 -> 34, bf16 all tangents H8 L1000 101 -> 180.  Not good enough for fp32 up to about 100 keys: the
        // fp32-MFMA kernel with 64 rows to a workgroup that was here before took, without tangents, H16 Lq600 Lkv77 24.6 us against
        // 32.3, all tangents H24 Lq4000 Lkv20 224 against 323 (but was half again as far from 64 bits).
        constexpr int KW = std::is_same<TIn, float>::value && TAN != TAN_NONE ? 2 : 1;
        int dev = 0, cus = 0;
        const hipError_t e = device_cus(&dev, &cus);
        if (e != hipSuccess) return e;
        auto cost = [&](int rows, int waves, double fixed) {
            const long long rounds = ((long long)((p.Lq - 1) / rows + 1) * p.B * p.H - 1) / cus + 1;
            return rounds * (fixed + ((p.Lkv - 1) / BC) / waves + 1);
        };
        if (cost(BR * 4 / KW, KW, KW == 1 ? 4.0 : 1.6) < 0.93 * cost(BR, 4, 1.2)) return launch_waves<TIn, D, TAN, KW>(p);
    }
    return launch_waves<TIn, D, TAN, 4>(p);
}

template <typename TIn, int D>
hipError_t launch_tan(const Problem& p) {
    if (!p.tq) return launch_one<TIn, D, TAN_NONE>(p);
    if (!p.tk) return launch_one<TIn, D, TAN_QUERY>(p);
    return launch_one<TIn, D, TAN_ALL>(p);
}

template <typename TIn>
hipError_t launch_dim(const Problem& p) {
    switch (p.d) {
        case 32: return launch_tan<TIn, 32>(p);
        case 64: return launch_tan<TIn, 64>(p);
        case 96: return launch_tan<TIn, 96>(p);
        case 128: return launch_tan<TIn, 128>(p);
        case 256: return launch_keysplit_256(p);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace
}  // namespace attn_jvp
