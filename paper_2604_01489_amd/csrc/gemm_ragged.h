// bf16 GEMM for operands the direct-to-LDS kernels do not take: rows that start at any 2-byte address, sizes and
// leading dimensions that are multiples of nothing, a result whose rows no 16-byte piece divides.
//
// The tile goes to LDS through registers, in the layouts of the main kernel (bf16_layout.h: 128-byte rows for
// an operand whose memory rows run along k, two 32-k images for the other kind), so that the fragment reads and the
// multiply are the main kernel's.  A lane moves 16 bytes per load whatever the address (global memory takes
// unaligned vector accesses); only the last K step of a block, where a chunk may hang over the end of a row and
// the row may be the operand's last, pulls such a chunk back inside its row and shifts the bytes into place.  Rows
// and columns beyond M and N are clamped, not masked: what they multiply into is never stored.
//
// What bounds it: the vector cache's look-ups.  A wave's 1 KB load from rows at odd elements is 56 of them (17 where the rows are
// aligned, 25 at 4-byte addresses): 1999 x 1537 x 2051, 208 blocks of 128 x 128, makes 1.24e7, 6.0e4 a CU of the 7.7e4 cycles that
// it is busy.  The matrix pipes are busy for 0.22 of those, the LDS for 0.22 without a bank conflict, and 0.24 of the waves'
// time is spent waiting for loads.  A CU holds two workgroups (four of the 64 x 64 tile), which cover each other's barriers
// and waits where a launch has that many: these 208 blocks are one on each of 208 CUs.
#pragma once
#include <type_traits>

#include "ge_device.h"
#include "ragged_layout.h"

namespace ge {

// The chunks of one operand that a lane brings in per 64-k step of a tile BX wide (ragged_layout.h).
template <int BX, bool STRIDED>
struct RaggedChunks {
    static constexpr int NL = BX / 32;
    int off[NL], offLast[NL];               // byte offset of each chunk from the step's first element: in any step, in the last
    int ld, left;                           // leading dimension; rows (columns) of the operand from the tile's first

    __device__ __forceinline__ void init(int ld_, int left_, int kLast, int w, int lane)
    {
        ld = ld_;
        left = left_;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab, sh;
            long long at;
            ragged_place<BX, STRIDED>(j, w, lane, r, c, slab);
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
    __device__ __forceinline__ void settle_last(int kLeft, int w, int lane, i32x4_t (&v)[NL]) const
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab, sh;
            long long at;
            ragged_place<BX, STRIDED>(j, w, lane, r, c, slab);
            ragged_last<STRIDED, 8>(r, c, ld, left, kLeft, at, sh);
            v[j] = shift_down_elements(v[j], sh);
        }
    }
    __device__ __forceinline__ static void store(GE_LDS char *stage, int w, int lane, const i32x4_t (&v)[NL])
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab;
            ragged_place<BX, STRIDED>(j, w, lane, r, c, slab);
            *(GE_LDS i32x4_t *)(stage + slab * 1024 + lane * 16) = v[j];
        }
    }
};

// A stored M x K or (TA) K x M, B stored K x N or (TB) N x K.  MODE: 0 fp32 partial sums of one K slice, 1 the run-time
// consumer chain with fp32 output, 2 with bf16 output.  Four waves in a 2 x 2 arrangement on a BT x BT tile.
template <int BT, bool TA, bool TB, int MODE>
__global__ void __launch_bounds__(256, 2)
gemm_bf16_ragged_kernel(const GemmParams p)
{
    constexpr int WT = BT / 2, T = WT / 16, STAGE = BT * 128, IMAGE32 = BT * 64;
    using ChunksA = RaggedChunks<BT, TA>;
    using ChunksB = RaggedChunks<BT, !TB>;
    // A stages 0 and 1, then B stages 0 and 1
    __shared__ __attribute__((aligned(1024))) char smem[4 * STAGE];
    GE_LDS char *const lds = (GE_LDS char *)smem;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w >> 1, wn = w & 1;
    const TileCoord tc = map_block(p);
    const int m0 = tc.tm * BT, n0 = tc.tn * BT;
    int kBegin = tc.s * p.kPerSlice;
    int kEnd = min(p.K, kBegin + p.kPerSlice);
    triangular_k_range(p, m0, BT, kBegin, kEnd);
    const int nk = (kEnd - kBegin + 63) / 64, kLast = kEnd - kBegin - (nk - 1) * 64;     // steps; k of the last one

    const char *gA = (const char *)p.A + 2 * ((long long)tc.b * p.strideA + (TA ? (long long)kBegin * p.lda + m0 : (long long)m0 * p.lda + kBegin));
    const char *gB = (const char *)p.B + 2 * ((long long)tc.b * p.strideB + (TB ? (long long)n0 * p.ldb + kBegin : (long long)kBegin * p.ldb + n0));
    const long long stepA = TA ? (long long)p.lda * 128 : 128, stepB = TB ? 128 : (long long)p.ldb * 128;

    ChunksA ca;
    ChunksB cb;
    ca.init(p.lda, p.M - m0, kLast, w, lane);
    cb.init(p.ldb, p.N - n0, kLast, w, lane);
    // two register sets: even steps travel in set 0 to LDS stage 0, odd ones in set 1 to stage 1.  Steps beyond the last
    // are the last one again, so that no load sits behind a branch (whose two sides the compiler joins by copying
    // the registers, which waits for the loads).
    i32x4_t va[2][ChunksA::NL], vb[2][ChunksB::NL];
    auto load = [&](int t, auto set) {
        constexpr int S = decltype(set)::value;
        const bool last = t + 1 >= nk;
        const int tt = last ? nk - 1 : t;
        ca.load(gA + tt * stepA, last, va[S]);
        cb.load(gB + tt * stepB, last, vb[S]);
    };
    auto store = [&](auto set) {
        constexpr int S = decltype(set)::value;
        ChunksA::store(lds + S * STAGE, w, lane, va[S]);
        ChunksB::store(lds + (2 + S) * STAGE, w, lane, vb[S]);
    };
    auto settle = [&](auto set) {
        constexpr int S = decltype(set)::value;
        ca.settle_last(kLast, w, lane, va[S]);
        cb.settle_last(kLast, w, lane, vb[S]);
    };
    auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // fragment addresses as in the main kernel: one base per k half of a 128-byte-row stage, one per 16-row block of
    // a k-strided one
    unsigned aAt[TA ? T : 2], bAt[TB ? 2 : T];
#pragma unroll
    for (int i = 0; i < (TA ? T : 2); ++i)
        aAt[i] = TA ? (unsigned)b_frag_offset<BT>(wm * WT, lane, 0) ^ (unsigned)(i * 32) : (unsigned)a64_frag_offset(wm * WT, lane, i);
#pragma unroll
    for (int j = 0; j < (TB ? 2 : T); ++j)
        bAt[j] = (unsigned)(2 * STAGE) + (TB ? (unsigned)a64_frag_offset(wn * WT, lane, j) : (unsigned)b_frag_offset<BT>(wn * WT, lane, 0) ^ (unsigned)(j * 32));
    auto read_strided = [&](unsigned at) {
        const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)(lds + at));
        const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)(lds + at + 4 * BT * 2));
        return __builtin_bit_cast(bf16x8_t, (short8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    f32x4_t acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

    auto multiply = [&](int s) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8_t fa[T], fb[T];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                if (TA) fa[i] = read_strided(aAt[TA ? i : 0] + (unsigned)(s * STAGE + h * IMAGE32));
                else fa[i] = *(const GE_LDS bf16x8_t *)(lds + aAt[TA ? 0 : h] + s * STAGE + i * 2048);
            }
#pragma unroll
            for (int j = 0; j < T; ++j) {
                if (TB) fb[j] = *(const GE_LDS bf16x8_t *)(lds + bAt[TB ? h : 0] + s * STAGE + j * 2048);
                else fb[j] = read_strided(bAt[TB ? 0 : j] + (unsigned)(s * STAGE + h * IMAGE32));
            }
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    if (MODE == 2) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
                    else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
                }
        }
    };

    // One barrier per step: step t writes the stage that step t - 1 read, from registers that memory was asked to fill two
    // steps ago, asks for step t + 3, and multiplies.  (One step ahead only, a workgroup alone on its CU waits for
    // memory in every step: 1999 x 1537 x 2051 on 208 tiles of 128 x 128 took 39 us.)
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    if (nk > 0) {
        load(0, S0{});
        load(1, S1{});
        if (nk == 1) settle(S0{});
        store(S0{});
        load(2, S0{});
        barrier();
        int t = 0;
        for (; t + 3 < nk; t += 2) {          // neither of the two steps written here is the last
            store(S1{});
            load(t + 3, S1{});
            multiply(0);
            barrier();
            store(S0{});
            load(t + 4, S0{});
            multiply(1);
            barrier();
        }
        // one, two or three steps are left, the first of them in stage 0
        const int left = nk - t;
        if (left > 1) {
            if (left == 2) settle(S1{});
            store(S1{});
        }
        multiply(0);
        if (left > 1) {
            barrier();
            if (left > 2) {
                settle(S0{});
                store(S0{});
            }
            multiply(1);
            if (left > 2) {
                barrier();
                multiply(0);
            }
        }
        barrier();
    }

    if constexpr (MODE == 2) {
        fused_epilogue_bf16_through_lds<BT, BT, 4, 4 * STAGE, T, T, true, false, true>(
            p, tc.b, acc, lds, m0, n0, wm * WT + (lane & 15), wn * WT + 4 * (lane >> 4), w, lane);
    } else {
        const int rowLane = m0 + wm * WT + 4 * (lane >> 4), colLane = n0 + wn * WT + (lane & 15);
        if constexpr (MODE == 1) {
            if (tile_inside(m0, BT, p.M) && tile_inside(n0, BT, p.N)) fused_epilogue_f32_direct<T, T, false>(p, tc.b, acc, rowLane, colLane);
            else fused_epilogue_f32_direct<T, T, true>(p, tc.b, acc, rowLane, colLane);
        } else {
            float *cBase = p.C + (long long)tc.s * p.sliceStride + (long long)tc.b * p.M * p.N;
            if (tile_inside(m0, BT, p.M) && tile_inside(n0, BT, p.N)) store_plain_tile<true, ACT_NONE, false>(nullptr, 1.0f, cBase, p.N, p.M, p.N, acc, rowLane, colLane);
            else store_plain_tile<true, ACT_NONE, true>(nullptr, 1.0f, cBase, p.N, p.M, p.N, acc, rowLane, colLane);
        }
    }
}

}  // namespace ge
