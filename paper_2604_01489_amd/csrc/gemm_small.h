// bf16 GEMM and convolution for few output tiles: 32 x 32 tiles, 256 k to a step, operands of any alignment.
//
// What bounds such a product on the larger tiles is neither bytes nor the matrix pipes: a block walks K alone on its CU, one barrier and
// one trip through LDS after the other (0.28 us for each 64 k of a 64 x 64 tile, of which the multiplies are 0.05), and most CUs have
// no block.  Small tiles give more CUs a block, and a step of 256 k pays for one barrier and one trip through LDS what the others pay four
// times, with two further steps on their way in registers.  Every wave multiplies one 16 x 16 block over all of K, in the order of the other
// kernels (the same bits); what the epilogue needs is asked for before the walk over K.
#pragma once
#include <type_traits>

#include "ge_device.h"
#include "small_layout.h"

namespace ge {

template <int BX, int NW, bool STRIDED>
struct SmallChunks {
    static constexpr int NL = small_chunks<BX, NW>();
    int off[NL], offLast[NL];               // byte offset of each chunk from the step's first element: in any step but the last, in the last
    int ld, left;

    __device__ __forceinline__ void init(int ld_, int left_, int kLast, int w, int lane)
    {
        ld = ld_;
        left = left_;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, place, sh;
            long long at;
            small_place<BX, NW, STRIDED>(j, w, lane, r, c, place);
            off[j] = (int)ragged_offset<STRIDED, 8>(r, c, ld, left) * 2;
            ragged_last<STRIDED, 8>(r, c, ld, left, kLast, at, sh);
            offLast[j] = (int)at * 2;
        }
    }
    __device__ __forceinline__ void load(const char *step, bool last, i32x4_t (&v)[NL]) const
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) v[j] = ((const i32x4_any_t *)(step + (last ? offLast[j] : off[j])))->v;
    }
    // what the last step read is put in its place when it has arrived
    __device__ __forceinline__ void settle_last(int kLast, int w, int lane, i32x4_t (&v)[NL]) const
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, place, sh;
            long long at;
            small_place<BX, NW, STRIDED>(j, w, lane, r, c, place);
            ragged_last<STRIDED, 8>(r, c, ld, left, kLast, at, sh);
            v[j] = shift_down_elements(v[j], sh);
        }
    }
    __device__ __forceinline__ static void store(GE_LDS char *stage, int w, int lane, const i32x4_t (&v)[NL])
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, place;
            small_place<BX, NW, STRIDED>(j, w, lane, r, c, place);
            *(GE_LDS i32x4_t *)(stage + place) = v[j];
        }
    }
};

// The gathered rows of a convolution in the same places: row r of the tile is an output position, a chunk eight channels of one filter tap (channels are a
// multiple of 8), the same ones for all of a lane's chunks.  Padding, positions beyond the last and k beyond the last read zeros, out of the resource's range.
template <int NW>
struct SmallConvRows {
    static constexpr int NL = small_chunks<32, NW>();
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
    int ih0[NL], iw0[NL], k0;               // input row and column of tap (0, 0); k of the lane's chunk in the first step
    unsigned off[NL];                       // byte offset of that element, modulo 2^32 (it may lie in the padding)
    buffer_t rows;

    __device__ __forceinline__ void init(const GemmParams &p, int m0, int w, int lane)
    {
        rows = __builtin_amdgcn_make_buffer_rsrc((void *)p.A, 0, (int)p.bytesA, 0x00020000);
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, place;
            small_place<32, NW, false>(j, w, lane, r, c, place);
            const int m = m0 + r, pos = m % (p.convOH * p.convOW), img = m / (p.convOH * p.convOW), oh = pos / p.convOW, ow = pos % p.convOW;
            const int row = oh * p.convSh - p.convPh;
            ih0[j] = m < p.M ? row : -(1 << 24);
            iw0[j] = ow * p.convSw - p.convPw;
            off[j] = (unsigned)((img * p.convH + row) * p.convW + iw0[j]) * (unsigned)p.convCin * 2u;
            k0 = c * 8;
        }
    }
    __device__ __forceinline__ void load(const GemmParams &p, int t, i32x4_t (&v)[NL]) const
    {
        const int k = t * SMALL_STEP + k0, tap = (int)((unsigned)k / (unsigned)p.convCin), kh = (int)((unsigned)tap / (unsigned)p.convKW);
        const int dIh = kh * p.convDh, dIw = (tap - kh * p.convKW) * p.convDw;
        const unsigned tapOff = (unsigned)(((dIh * p.convW + dIw) * p.convCin + (k - tap * p.convCin)) * 2);
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const bool inside = k < p.K && (unsigned)(ih0[j] + dIh) < (unsigned)p.convH && (unsigned)(iw0[j] + dIw) < (unsigned)p.convW;
            v[j] = __builtin_bit_cast(i32x4_t, (u32x4_t)__builtin_amdgcn_raw_buffer_load_b128(rows, (int)(inside ? off[j] + tapOff : 0x80000000u), 0, 0));
        }
    }
};

// A stored M x K or (TA) K x M, or (CONV) the gathered rows of a convolution, B stored K x N or (TB) N x K; the run-time consumer chain with fp32 or (OUTBF16) bf16 output.  run: steps
// whose sums form one chain (small_run).
// DEPTH: steps on their way in registers (one: K is one step at most).
template <int DEPTH, bool TA, bool TB, bool OUTBF16, bool CONV = false>
__global__ void __launch_bounds__(256)
gemm_bf16_small_kernel(const GemmParams p, int run)
{
    constexpr int BM = 32, BN = 32, NW = 4, WN = 2, STAGE_A = BM * 512, STAGE_B = BN * 512, STAGES = DEPTH == 1 ? 1 : 2;
    static_assert(!CONV || (!TA && TB), "rows along k, filters as N x K");
    using ChunksA = SmallChunks<BM, NW, TA>;
    using ChunksB = SmallChunks<BN, NW, !TB>;
    __shared__ __attribute__((aligned(1024))) char smem[STAGES * (STAGE_A + STAGE_B)];
    GE_LDS char *const lds = (GE_LDS char *)smem;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w / WN, wn = w % WN;
    const TileCoord tc = map_block(p);
    const int m0 = tc.tm * BM, n0 = tc.tn * BN;
    const int nk = (p.K + SMALL_STEP - 1) / SMALL_STEP, kLast = p.K - (nk - 1) * SMALL_STEP;

    const char *gA = (const char *)p.A + 2 * ((long long)tc.b * p.strideA + (TA ? (long long)m0 : (long long)m0 * p.lda));
    const char *gB = (const char *)p.B + 2 * ((long long)tc.b * p.strideB + (TB ? (long long)n0 * p.ldb : (long long)n0));
    const long long stepA = (TA ? (long long)p.lda : 1ll) * SMALL_STEP * 2, stepB = (TB ? 1ll : (long long)p.ldb) * SMALL_STEP * 2;
    std::conditional_t<CONV, SmallConvRows<NW>, ChunksA> ca;
    ChunksB cb;
    if constexpr (CONV) ca.init(p, m0, w, lane);
    else ca.init(p.lda, p.M - m0, kLast, w, lane);
    cb.init(p.ldb, p.N - n0, kLast, w, lane);
    i32x4_t va[DEPTH][ChunksA::NL], vb[DEPTH][ChunksB::NL];
    // (steps beyond the last are the last one again: no load behind a branch)
    auto load = [&](int t, auto set) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        const bool last = t + 1 >= nk;
        const int tt = last ? nk - 1 : t;
        if constexpr (CONV) ca.load(p, tt, va[S]);
        else ca.load(gA + tt * stepA, last, va[S]);
        cb.load(gB + tt * stepB, last, vb[S]);
    };
    auto store = [&](auto set, bool last) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        if (last) {
            if constexpr (!CONV) ca.settle_last(kLast, w, lane, va[S]);
            cb.settle_last(kLast, w, lane, vb[S]);
        }
        ChunksA::store(lds + S % STAGES * STAGE_A, w, lane, va[S]);
        ChunksB::store(lds + STAGES * STAGE_A + S % STAGES * STAGE_B, w, lane, vb[S]);
    };
    auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // f(0), f(1), .. f(DEPTH - 1)
    auto each = [&](auto f) __attribute__((always_inline)) {
        f(std::integral_constant<int, 0>{});
        if constexpr (DEPTH > 1) f(std::integral_constant<int, 1 % DEPTH>{});
    };
    static_assert(DEPTH == 1 || DEPTH == 2, "sets of registers");
    each([&](auto set) __attribute__((always_inline)) { load(decltype(set)::value, set); });

    // What the epilogue needs.  fp32: register r of a lane is row 4 (l / 16) + r, column l % 16 of the wave's block; bf16 (operands
    // of the multiply swapped): row l % 16, column 4 (l / 16) + r.  Beyond M and N: the last row's and column's, which are never stored.
    const int mLane = m0 + wm * 16 + (OUTBF16 ? lane & 15 : 4 * (lane >> 4)), nLane = n0 + wn * 16 + (OUTBF16 ? 4 * (lane >> 4) : lane & 15);
    // Nothing is computed from it here, and the residual's type is branched on once for all four: a conversion waits for its load, and for the operands' on their way before
    // it (a bf16 residual element by element was four round trips to memory before the walk: A K x M, B N x K, fp32 out, 199 x 465 x 273 6.5 -> 5.9 us, 256 x 512 x 512 5.5 -> 5.0).
    float rowScale[4], bias[4];
    unsigned raw[4] = {0u, 0u, 0u, 0u};
    int mAt[4], nAt[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        mAt[r] = OUTBF16 ? min(mLane, p.M - 1) : min(mLane + r, p.M - 1);
        nAt[r] = OUTBF16 ? min(nLane + r, p.N - 1) : min(nLane, p.N - 1);
        rowScale[r] = p.rowScale != nullptr ? p.rowScale[mAt[r]] : 1.0f;
        bias[r] = p.bias != nullptr ? p.bias[nAt[r]] : 0.0f;
    }
    const bool resBf16 = p.rType == DT_BF16;
    if (p.R != nullptr) {
        const long long rBase = (long long)tc.b * p.strideR;
        if (resBf16) {
#pragma unroll
            for (int r = 0; r < 4; ++r) raw[r] = ((const unsigned short *)p.R)[rBase + (long long)mAt[r] * p.ldr + nAt[r]];
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) raw[r] = ((const unsigned *)p.R)[rBase + (long long)mAt[r] * p.ldr + nAt[r]];
        }
    }

    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f}, sum = acc;       // of this run of steps, of the runs before it
    int inRun = 0;
    const int aAt = TA ? b_frag_offset<BM>(wm * 16, lane, 0) : 0, bAt = TB ? 0 : b_frag_offset<BN>(wn * 16, lane, 0);
    auto read_strided = [&](const GE_LDS char *at, int rowBytes) __attribute__((always_inline)) {
        const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)at);
        const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)(at + 4 * rowBytes));
        return __builtin_bit_cast(bf16x8_t, (short8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto multiply = [&](auto set) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value % STAGES;
        const GE_LDS char *const sA = lds + S * STAGE_A, *const sB = lds + STAGES * STAGE_A + S * STAGE_B;
        if (inRun == run) {
#pragma unroll
            for (int r = 0; r < 4; ++r) { sum[r] += acc[r]; acc[r] = 0.0f; }
            inRun = 0;
        }
        ++inRun;
        bf16x8_t fa[8], fb[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if constexpr (TA) fa[q] = read_strided(sA + aAt + q * (BM * 64), BM * 2);
            else fa[q] = *(const GE_LDS bf16x8_t *)(sA + a64_frag_offset(wm * 16, lane, q & 1) + (q >> 1) * (BM * 128));
            if constexpr (TB) fb[q] = *(const GE_LDS bf16x8_t *)(sB + a64_frag_offset(wn * 16, lane, q & 1) + (q >> 1) * (BN * 128));
            else fb[q] = read_strided(sB + bAt + q * (BN * 64), BN * 2);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (OUTBF16) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[q], fa[q], acc, 0, 0, 0);
            else acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[q], fb[q], acc, 0, 0, 0);
        }
    };

    // One barrier per step: step t writes the stage that step t - 1 read, from registers that memory was asked to fill DEPTH steps ago,
    // asks for the step as far ahead, and multiplies.
    using S0 = std::integral_constant<int, 0>;
    store(S0{}, nk == 1);
    if constexpr (DEPTH == 1) {
        barrier();
        multiply(S0{});
    } else {
        load(DEPTH, S0{});
        barrier();
        int t = 0;
        for (; t + DEPTH + 1 < nk; t += DEPTH)               // none of the steps written here is the last
            each([&](auto set) __attribute__((always_inline)) {
                constexpr int U = decltype(set)::value;
                using Next = std::integral_constant<int, (U + 1) % DEPTH>;
                store(Next{}, false);
                load(t + U + 1 + DEPTH, Next{});
                multiply(set);
                barrier();
            });
        // one to DEPTH + 1 steps are left, the first of them in stage 0
        const int left = nk - t;
        each([&](auto set) __attribute__((always_inline)) {
            constexpr int U = decltype(set)::value;
            if (U < left) {
                if (U + 1 < left) store(std::integral_constant<int, (U + 1) % DEPTH>{}, U + 2 == left);
                multiply(set);
                if (U + 1 < left) barrier();
            }
        });
        if (left == DEPTH + 1) multiply(S0{});
    }

    if (nk > run) {
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = sum[r] + acc[r];
    }
    f32x4_t v[1];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[0][r] = __builtin_fmaf(acc[r], p.alpha * rowScale[r], bias[r]);
    if (p.R != nullptr) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[0][r] = __builtin_fmaf(p.beta, __uint_as_float(resBf16 ? raw[r] << 16 : raw[r]), v[0][r]);
    }
    act_clamp_row_block<1>(p, v);
    if constexpr (OUTBF16) {
        if (mLane >= p.M) return;
        unsigned short *dst = (unsigned short *)p.C + (long long)tc.b * p.strideC + (long long)mLane * p.ldc + nLane;
        u32x2_t o;
        o[0] = pack_bf16_pair(v[0][0], v[0][1]);
        o[1] = pack_bf16_pair(v[0][2], v[0][3]);
        if (nLane + 4 <= p.N) ((u32x2_any_t *)dst)->v = o;
        else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (nLane + e < p.N) dst[e] = (unsigned short)(o[e >> 1] >> (16 * (e & 1)));
        }
    } else {
        float *dst = p.C + (long long)tc.b * p.strideC + (long long)mLane * p.ldc + nLane;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (mLane + r < p.M && nLane < p.N) dst[(long long)r * p.ldc] = v[0][r];
    }
}

}  // namespace ge
