// fp32 matrix-core streaming kernel for attention forward + JVP (paper App. C.1, Alg. 2) at head dimension 256, fp32 or
// bf16 inputs (upcast exactly), every product and sum in fp32.
//
// Two tensors of 256 columns (the accumulators) and two of 256 elements per query row (Q, tQ) do not fit the registers
// of a wave that owns 32 rows, so the kernels for smaller head dimensions do not extend to this one.  Here a wave owns 16
// rows and all six products run on v_mfma_f32_16x16x4_f32, transposed as in those kernels: S^T = K Q^T, O^T += V^T P~^T,
// query = MFMA column (lane % 16).  With gg = lane / 16, a lane holds the scores of keys 4 gg .. 4 gg + 3 of its query,
// which are the B operands of the four reduction steps of the value products as they stand.
//   score step (u, e), u < 16, e < 4: A = K[key = lane % 16][16 u + 4 gg + e], B = Q[query = lane % 16][16 u + 4 gg + e]
//   value step r < 4, columns (cq, e): A = V[key 4 gg + r][64 cq + 4 (lane % 16) + e], B = weight register r
// so every operand comes from LDS as part of a 16-byte read; chunk c of row j sits at c ^ j, which spreads the reads of
// sixteen rows, and of sixteen neighbouring chunks, over all banks.  Blocks of 16 keys are fetched into registers one
// block ahead and written (upcast) into the other of two LDS stages.  The scores are
// summed over groups of 16 elements (four MFMAs), and these in a tree: one chain of 256 elements would carry twice the
// rounding error.
//
// Bound by the fp32 matrix pipe (384 MFMAs of 32 cycles per wave and block; nothing of it overlaps with vector work):
// B1 H4 L3000, all tangents: 1.6 ms = 69 TFLOP/s counted with 188 workgroups (10.4 ms on the vector ALU, sixteen lanes to a
// row); B2 H8 Lq4000 Lkv300 without key tangents 0.49 ms (3.9).  Errors against 64 bits as there.
#include "launchers.h"
#include <hip/hip_bf16.h>
#include <type_traits>

namespace attn_jvp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 256, BR = 64, BC = 16, NTHREADS = 256;
constexpr int CH = D / 4;                    // 16-byte chunks of an fp32 row
constexpr int TAN_NONE = 0, TAN_QUERY = 1, TAN_ALL = 2;
// Nats by which a row's scores may exceed m before m is moved.  The weights are exp(S - (m + MAX_SLACK)), never above 1, so that
// values up to the end of the fp32 range stay in it; the price, weights that flush to zero MAX_SLACK nats earlier, is why
// there are few.
constexpr float MAX_SLACK = 4.f;

template <typename T> struct In;             // four consecutive elements as they are in memory, and upcast
template <> struct In<float> {
    typedef f32x4 Raw;
    static __device__ __forceinline__ f32x4 up(Raw r) { return r; }
};
template <> struct In<__hip_bfloat16> {
    typedef uint32_t Raw __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ f32x4 up(Raw r) {
        return f32x4{__uint_as_float(r[0] << 16), __uint_as_float(r[0] & 0xffff0000u),
                     __uint_as_float(r[1] << 16), __uint_as_float(r[1] & 0xffff0000u)};
    }
};
__device__ __forceinline__ void store4(float* p, f32x4 x) { *reinterpret_cast<f32x4*>(p) = x; }
__device__ __forceinline__ void store4(__hip_bfloat16* p, f32x4 x) {
    alignas(8) __hip_bfloat16 h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = __float2bfloat16(x[i]);
    *reinterpret_cast<uint2*>(p) = *reinterpret_cast<const uint2*>(h);
}
__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <typename TIn, typename TOut, int TAN>
__global__ __launch_bounds__(NTHREADS, 1) void attn_jvp_fp32_d256_kernel(
    const TIn* __restrict__ Q, const TIn* __restrict__ K, const TIn* __restrict__ V,
    const TIn* __restrict__ tQ, const TIn* __restrict__ tK, const TIn* __restrict__ tV,
    TOut* __restrict__ O, TOut* __restrict__ tO, float* __restrict__ LSE,
    int Lq, int Lkv, float scale, int q_tiles, int H, int blhd) {
    // (the instantiations must agree bit for bit, absent tangents against zero ones: no implicit fusing)
#pragma clang fp contract(off)
    constexpr bool TANGENT = TAN != TAN_NONE, KV_TANGENT = TAN == TAN_ALL;
    constexpr int NT = KV_TANGENT ? 4 : 2;           // K, V (, tK, tV)
    constexpr int PT = BC * CH / NTHREADS;           // chunks a lane moves per tensor and block
    typedef typename In<TIn>::Raw Raw;
    extern __shared__ f32x4 smem[];                  // [2 stages][NT][BC * CH]
    auto tile = [&](int stage, int x) { return smem + (stage * NT + x) * (BC * CH); };

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, gg = lane >> 4;
    // workgroups go round-robin over the 8 XCDs: a contiguous range of tiles for each, so that they share their keys in L2
    const int n_wg = gridDim.x;
    const int bid = (n_wg & 7) == 0 ? (int)(blockIdx.x & 7) * (n_wg >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const long bh = bid / q_tiles;
    const int qrow = (bid % q_tiles) * BR + 16 * wave + j;
    const int qload = qrow < Lq ? qrow : Lq - 1;     // rows past the end repeat the last one and are not stored
    // [B,H,L,d]: rows of a head contiguous; [B,L,H,d]: rows of a head H*d elements apart
    const long row_elems = blhd ? (long)H * D : D;
    const long bidx = bh / H, hidx = bh % H;
    const long q_base = blhd ? (bidx * Lq * H + hidx) * D : bh * (long)Lq * D;
    const long kv_base = blhd ? (bidx * Lkv * H + hidx) * D : bh * (long)Lkv * D;

    f32x4 q[16], tq[TANGENT ? 16 : 1];               // elements 16 u + 4 gg .. + 3 of the lane's row
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const long at = q_base + (long)qload * row_elems + 16 * u + 4 * gg;
        q[u] = In<TIn>::up(*reinterpret_cast<const Raw*>(Q + at));
        if constexpr (TANGENT) tq[u] = In<TIn>::up(*reinterpret_cast<const Raw*>(tQ + at));
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {                   // only MFMAs read them: keep them in accumulation registers
        asm volatile("" : "+a"(q[u]));
        if constexpr (TANGENT) asm volatile("" : "+a"(tq[u]));
    }

    // chunk n of a tensor's block that this lane moves: row wave + 4 n, chunk `lane` (rows past the end: the last key again)
    Raw stage_raw[NT][PT];
    auto fetch = [&](int blk) __attribute__((always_inline)) {
        const TIn* xs[4] = {K, V, tK, tV};
#pragma unroll
        for (int x = 0; x < NT; ++x)
#pragma unroll
            for (int n = 0; n < PT; ++n) {
                int row = blk * BC + wave + 4 * n;
                row = row < Lkv ? row : Lkv - 1;
                stage_raw[x][n] = *reinterpret_cast<const Raw*>(xs[x] + kv_base + (long)row * row_elems + 4 * lane);
            }
    };
    auto publish = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < NT; ++x)
#pragma unroll
            for (int n = 0; n < PT; ++n) tile(stage, x)[(wave + 4 * n) * CH + (lane ^ (wave + 4 * n))] = In<TIn>::up(stage_raw[x][n]);
    };

    f32x4 acc_o[16], acc_t[TANGENT ? 16 : 1];        // [4 cq + e][r]: column 64 cq + 4 (4 gg + r) + e
#pragma unroll
    for (int n = 0; n < 16; ++n) {
        acc_o[n] = f32x4{};
        if constexpr (TANGENT) acc_t[n] = f32x4{};
    }
    float m = -INFINITY, row_top = -INFINITY, l = 0.f, r_sum = 0.f;       // l, r: this lane's keys only, the four lanes of a row meet in the epilogue
    const int n_blocks = (Lkv + BC - 1) / BC;
    fetch(0);
    publish(0);
    __syncthreads();
    // (no instruction: keeps the accumulators in accumulation registers where the vector ALU does not read them)
    auto pin = [&](f32x4& a, f32x4& t) __attribute__((always_inline)) {
        asm volatile("" : "+a"(a));
        if constexpr (TANGENT) asm volatile("" : "+a"(t));
    };
    for (int blk = 0; blk < n_blocks; ++blk) {
        const int cur = blk & 1;
#pragma unroll
        for (int n = 0; n < 16; ++n) pin(acc_o[n], acc_t[TANGENT ? n : 0]);
        if (blk + 1 < n_blocks) fetch(blk + 1);
        // ---- S^T = K Q^T, tS^T = K tQ^T + tK Q^T
        const f32x4* lk = tile(cur, 0) + j * CH;
        f32x4 s_part[5], ts_part[TANGENT ? 5 : 1];   // sums over 1, 2, 4, 8, 16 groups of 16 elements: a binary counter
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const f32x4 ka = lk[(4 * u + gg) ^ j];
            f32x4 tka = ka;
            if constexpr (KV_TANGENT) tka = lk[2 * BC * CH + ((4 * u + gg) ^ j)];
            f32x4 su = {}, tu = {};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                su = mfma(ka[e], q[u][e], su);
                if constexpr (TANGENT) tu = mfma(ka[e], tq[u][e], tu);
            }
            if constexpr (KV_TANGENT)
#pragma unroll
                for (int e = 0; e < 4; ++e) tu = mfma(tka[e], q[u][e], tu);
            int level = 0;
#pragma unroll
            for (int b = u; b & 1; b >>= 1, ++level) {
                su = s_part[level] + su;
                if constexpr (TANGENT) tu = ts_part[level] + tu;
            }
            s_part[level] = su;
            if constexpr (TANGENT) ts_part[level] = tu;
        }
        const f32x4 s = s_part[4], ts = ts_part[TANGENT ? 4 : 0];
        // ---- online softmax on the lane's four keys; m trails the row maximum by up to MAX_SLACK
        float mb = -INFINITY;
        bool dead[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dead[r] = blk * BC + 4 * gg + r >= Lkv;
            mb = fmaxf(mb, dead[r] ? -INFINITY : s[r] * scale);
        }
        mb = fmaxf(mb, __shfl_xor(mb, 16));
        mb = fmaxf(mb, __shfl_xor(mb, 32));
        row_top = fmaxf(row_top, mb);                // the maximum itself, for lse: m + log l would round twice as often
        const float m_new = mb > m + MAX_SLACK ? mb : m;
        const float alpha = m_new == m ? 1.f : expf(m - m_new);         // 0 when the first finite score comes (m = -inf)
        m = m_new;
        const float m_ref = m == -INFINITY ? 0.f : m + MAX_SLACK;       // (scores of -inf so far: weight 0, not NaN)
        if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
            for (int n = 0; n < 16; ++n) {
                pin(acc_o[n], acc_t[TANGENT ? n : 0]);
                acc_o[n] *= alpha;
                if constexpr (TANGENT) acc_t[n] *= alpha;
                pin(acc_o[n], acc_t[TANGENT ? n : 0]);
            }
        }
        float p[4], h[4], row_p = 0.f, row_h = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = dead[r] ? 0.f : expf(fmaf(s[r], scale, -m_ref));
            row_p += p[r];
            h[r] = TANGENT && !dead[r] ? p[r] * (ts[r] * scale) : 0.f;
            row_h += h[r];
        }
        l = fmaf(alpha, l, row_p);
        r_sum = fmaf(alpha, r_sum, row_h);
        // ---- O^T += V^T P~^T, (A+B)^T += V^T H~^T + tV^T P~^T
        const f32x4* lv = tile(cur, 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 4 * gg + r;
#pragma unroll
            for (int cq = 0; cq < 4; ++cq) {
                const f32x4 va = lv[row * CH + ((16 * cq + j) ^ row)];
                f32x4 tva = va;
                if constexpr (KV_TANGENT) tva = lv[2 * BC * CH + row * CH + ((16 * cq + j) ^ row)];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc_o[4 * cq + e] = mfma(va[e], p[r], acc_o[4 * cq + e]);
                    if constexpr (TANGENT) acc_t[4 * cq + e] = mfma(va[e], h[r], acc_t[4 * cq + e]);
                }
                if constexpr (KV_TANGENT)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc_t[4 * cq + e] = mfma(tva[e], p[r], acc_t[4 * cq + e]);
            }
        }
        if (blk + 1 < n_blocks) publish(cur ^ 1);
        __syncthreads();     // next stage written by all, this stage read by all
    }

    float l_row = l + __shfl_xor(l, 16), r_row = r_sum + __shfl_xor(r_sum, 16);
    l_row += __shfl_xor(l_row, 32);
    r_row += __shfl_xor(r_row, 32);
    if (qrow < Lq) {
        const float inv_l = 1.f / l_row;
        const float mu = r_row * inv_l;              // rowsum(P o tS)
        TOut* op = O + q_base + (long)qrow * row_elems + 16 * gg;
        TOut* top = TANGENT ? tO + q_base + (long)qrow * row_elems + 16 * gg : nullptr;
#pragma unroll
        for (int cq = 0; cq < 4; ++cq)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                f32x4 o4, t4;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float o = acc_o[4 * cq + e][r];
                    if constexpr (TANGENT) t4[e] = fmaf(-mu, o, acc_t[4 * cq + e][r]) * inv_l;
                    o4[e] = o * inv_l;
                }
                store4(op + 64 * cq + 4 * r, o4);
                if constexpr (TANGENT) store4(top + 64 * cq + 4 * r, t4);
            }
        if (gg == 0) LSE[bh * Lq + qrow] = row_top + logf(l_row * expf(m + MAX_SLACK - row_top));
    }
}

template <typename TIn, typename TOut, int TAN>
hipError_t launch_one(const Problem& p) {
    const int q_tiles = (p.Lq + BR - 1) / BR;
    const long long blocks = (long long)q_tiles * p.B * p.H;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    constexpr int smem = 2 * (TAN == TAN_ALL ? 4 : 2) * BC * D * (int)sizeof(float);
    auto kern = attn_jvp_fp32_d256_kernel<TIn, TOut, TAN>;
    int dev = 0, cus = 0;
    hipError_t e = device_cus(&dev, &cus);
    if (e == hipSuccess) e = ensure_dynamic_lds(reinterpret_cast<const void*>(kern), smem, dev);
    if (e != hipSuccess) return e;
    MainKernelTimer timer(p);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(NTHREADS), smem, p.stream,
                       (const TIn*)p.q, (const TIn*)p.k, (const TIn*)p.v, (const TIn*)p.tq, (const TIn*)p.tk, (const TIn*)p.tv,
                       (TOut*)p.o, (TOut*)p.to, p.lse, p.Lq, p.Lkv, p.scale, q_tiles, p.H, p.layout);
    return timer.finish(hipGetLastError());
}

template <typename TIn, typename TOut>
hipError_t launch_tan(const Problem& p) {
    if (!p.tq) return launch_one<TIn, TOut, TAN_NONE>(p);
    if (!p.tk) return launch_one<TIn, TOut, TAN_QUERY>(p);
    return launch_one<TIn, TOut, TAN_ALL>(p);
}

}  // namespace

hipError_t launch_fp32_d256(const Problem& p) {
    if (p.d != D) return hipErrorInvalidValue;
    if (p.in_dtype == 1) return launch_tan<float, float>(p);                      // fp32 in -> fp32 out either way
    if (p.out_dtype == 0) return launch_tan<__hip_bfloat16, float>(p);
    return launch_tan<__hip_bfloat16, __hip_bfloat16>(p);
}

}  // namespace attn_jvp
