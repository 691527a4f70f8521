// fp32 GEMM for few output tiles, operands of any alignment: 32 x 32 tiles of which each wave multiplies a 16 x 16 block, or 16 x 16 tiles
// whose four waves share K.
//
// What bounds such a product on the 64 x 64 tiles is a block's walk over K alone on its CU, 0.6 us for each 32 k, while most CUs have no
// block.  Small tiles give more CUs one, and a step of 128 (256) k pays for one barrier and one trip through LDS, with two further
// steps on their way in registers; the matrix pipe takes 0.43 us for such a step of a 32 x 32 tile, a quarter of it for 128 k of a 16 x 16 one.
// v_mfma_f32_16x16x4_f32: which k a lane's operand is does not matter as long as A and B agree, so a lane takes four
// neighbouring k of its row of A with one 16-byte read.  LDS rows are padded so that a wave's reads fall in different banks.  Which products come
// here, and their times on either side: small_layout.h (few_tile_f32).
#pragma once
#include <type_traits>

#include "ge_device.h"
#include "small_layout.h"

namespace ge {

struct __attribute__((packed, aligned(4))) f32x4_few_t { f32x4_t v; };

template <int BT, bool STRIDED>
struct FewChunksF32 {
    int off[4], offLast[4];                 // byte offset of each chunk from the step's first element: in any step but the last, in the last
    int ld, left;

    __device__ __forceinline__ void init(int ld_, int left_, int kLast, int w, int lane)
    {
        ld = ld_;
        left = left_;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int r, c, place, sh;
            long long at;
            few_place_f32<BT, STRIDED>(j, w, lane, r, c, place);
            off[j] = (int)ragged_offset<STRIDED, 4>(r, c, ld, left) * 4;
            ragged_last<STRIDED, 4>(r, c, ld, left, kLast, at, sh);
            offLast[j] = (int)at * 4;
        }
    }
    __device__ __forceinline__ void load(const char *step, bool last, f32x4_t (&v)[4]) const
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = ((const f32x4_few_t *)(step + (last ? offLast[j] : off[j])))->v;
    }
    // what the last step read is put in its place when it has arrived
    __device__ __forceinline__ void settle_last(int kLast, int w, int lane, f32x4_t (&v)[4]) const
    {
        const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int r, c, place, sh;
            long long at;
            few_place_f32<BT, STRIDED>(j, w, lane, r, c, place);
            ragged_last<STRIDED, 4>(r, c, ld, left, kLast, at, sh);
            f32x4_t t = v[j];
            t = sh & 1 ? __builtin_shufflevector(t, zero, 1, 2, 3, 4) : t;
            t = sh & 2 ? __builtin_shufflevector(t, zero, 2, 3, 4, 4) : t;
            v[j] = sh >= 4 ? zero : t;
        }
    }
    __device__ __forceinline__ static void store(GE_LDS char *stage, int w, int lane, const f32x4_t (&v)[4])
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int r, c, place;
            few_place_f32<BT, STRIDED>(j, w, lane, r, c, place);
            *(GE_LDS f32x4_t *)(stage + place) = v[j];
        }
    }
};

// DEPTH: steps on their way in registers (one: K is one step at most)
template <int BT, int DEPTH>
__global__ void __launch_bounds__(256)
gemm_f32_few_kernel(const GemmParams p)
{
    constexpr int STEP = few_step_f32(BT), STAGES = DEPTH == 1 ? 1 : 2, STAGE_A = BT * few_pitch_a(BT), STAGE_B = STEP * few_pitch_b(BT);
    constexpr int KG = BT == 16 ? 4 : 1, GROUPS = STEP / KG / 16;              // waves that share K; 16-k groups of a step for a wave
    using ChunksA = FewChunksF32<BT, false>;
    using ChunksB = FewChunksF32<BT, true>;
    __shared__ __attribute__((aligned(1024))) char smem[STAGES * (STAGE_A + STAGE_B) + (KG > 1 ? KG * 1024 : 0)];
    GE_LDS char *const lds = (GE_LDS char *)smem;
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = KG > 1 ? 0 : w >> 1, wn = KG > 1 ? 0 : w & 1, kw = KG > 1 ? w * (STEP / KG) : 0;
    const TileCoord tc = map_block(p);
    const int m0 = tc.tm * BT, n0 = tc.tn * BT;
    const int nk = (p.K + STEP - 1) / STEP, kLast = p.K - (nk - 1) * STEP;

    const char *gA = (const char *)p.A + 4 * ((long long)tc.b * p.strideA + (long long)m0 * p.lda);
    const char *gB = (const char *)p.B + 4 * ((long long)tc.b * p.strideB + n0);
    const long long stepB = (long long)p.ldb * (STEP * 4);
    ChunksA ca;
    ChunksB cb;
    ca.init(p.lda, p.M - m0, kLast, w, lane);
    cb.init(p.ldb, p.N - n0, kLast, w, lane);
    f32x4_t va[DEPTH][4], vb[DEPTH][4];
    // (steps beyond the last are the last one again: no load behind a branch)
    auto load = [&](int t, auto set) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        const bool last = t + 1 >= nk;
        const int tt = last ? nk - 1 : t;
        ca.load(gA + tt * (STEP * 4ll), last, va[S]);
        cb.load(gB + tt * stepB, last, vb[S]);
    };
    auto store = [&](auto set, bool last) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        if (last) {
            ca.settle_last(kLast, w, lane, va[S]);
            cb.settle_last(kLast, w, lane, vb[S]);
        }
        ChunksA::store(lds + S * STAGE_A, w, lane, va[S]);
        ChunksB::store(lds + STAGES * STAGE_A + S * STAGE_B, w, lane, vb[S]);
    };
    auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, STAGES - 1>;
    load(0, S0{});
    if constexpr (DEPTH > 1) load(1, S1{});

    // the lane's column of C, and its bias (beyond N: the last column's, which is never stored)
    const int n = n0 + wn * 16 + l16;
    const float bias = p.bias != nullptr ? p.bias[min(n, p.N - 1)] : 0.0f;

    // a block's sums in four chains, as the waves that share K have them: the error of one is twice as large (512^3 4.1e-7 against 2.0e-7)
    constexpr int CHAINS = KG > 1 ? 1 : 4;
    f32x4_t acc[CHAINS];
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[c][r] = 0.0f;
    const int aAt = few_at_a(BT, wm * 16 + l16, kw + 4 * g), bAt = STAGES * STAGE_A + few_at_b(BT, kw + 4 * g, wn * 16 + l16);
    auto group = [&](int at, int q) __attribute__((always_inline)) {
        const f32x4_t a = *(const GE_LDS f32x4_t *)(lds + aAt + at * STAGE_A + q * 64);
        float b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = *(const GE_LDS float *)(lds + bAt + at * STAGE_B + (q * 16 + e) * few_pitch_b(BT));
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[q % CHAINS] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc[q % CHAINS], 0, 0, 0);
    };
    auto multiply = [&](auto set) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) group(decltype(set)::value, q);
    };
    // the last step: the groups that K reaches
    auto multiply_last = [&](auto set) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < GROUPS; ++q)
            if (kw + q * 16 < kLast) group(decltype(set)::value, q);
    };

    // One barrier per step: step t writes the stage that step t - 1 read, from registers that memory was asked to fill two
    // steps ago, asks for step t + 3, and multiplies.
    store(S0{}, nk == 1);
    if constexpr (DEPTH == 1) {
        barrier();
        multiply_last(S0{});
    } else {
        load(2, S0{});
        barrier();
        int t = 0;
        for (; t + 3 < nk; t += 2) {          // neither of the two steps written here is the last
            store(S1{}, false);
            load(t + 3, S1{});
            multiply(S0{});
            barrier();
            store(S0{}, false);
            load(t + 4, S0{});
            multiply(S1{});
            barrier();
        }
        // two or three steps are left (K is longer than one), the first of them in stage 0
        const int left = nk - t;
        store(S1{}, left == 2);
        multiply(S0{});
        barrier();
        if (left > 2) {
            store(S0{}, true);
            multiply(S1{});
            barrier();
            multiply_last(S0{});
        } else {
            multiply_last(S1{});
        }
    }

    // register r of a lane: row 4 (l / 16) + r of the wave's block
    float *dst = p.C + (long long)tc.b * p.strideC + n;
    if constexpr (KG == 1) {
        const int m = m0 + wm * 16 + 4 * g;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float v = acc[0][r];
#pragma unroll
            for (int c = 1; c < CHAINS; ++c) v += acc[c][r];
            if (m + r < p.M && n < p.N) dst[(long long)(m + r) * p.ldc] = epilogue_value_rt(v, p.alpha, bias, p.act);
        }
    } else {
        GE_LDS char *const sums = lds + STAGES * (STAGE_A + STAGE_B);         // [wave][lane]
        *(GE_LDS f32x4_t *)(sums + w * 1024 + lane * 16) = acc[0];
        barrier();
        float v = *(const GE_LDS float *)(sums + lane * 16 + w * 4);          // wave w: register w of every lane, the waves' sums in order
#pragma unroll
        for (int i = 1; i < KG; ++i) v += *(const GE_LDS float *)(sums + i * 1024 + lane * 16 + w * 4);
        const int m = m0 + 4 * g + w;
        if (m < p.M && n < p.N) dst[(long long)m * p.ldc] = epilogue_value_rt(v, p.alpha, bias, p.act);
    }
}

}  // namespace ge
