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
// What bounds it: the vector cache's look-ups, and a tile's phases where it is alone on its CU.  A wave's 1 KB load from rows at odd
// elements is 56 look-ups (17 where the rows are aligned, 25 at 4-byte addresses).  With eight waves to a 128 x 128 tile such rows are read
// from their second element on, at 4-byte addresses, and moved up by one behind the end of the neighbouring lane's chunk (one
// DPP move and four v_perm_b32 a chunk); the first element of each row comes by a 2-byte load.  1999 x 1537 x 2051, 208 blocks: 1.24e7 look-ups
// -> 7.1e6, and two waves on each SIMD that cover each other's waits: 33.8 -> 31.5 us (aligned rows, 1999 x 1540 x 2052, where
// only the waves tell: 27.9 -> 27.5); 1999 x 1537 x 4099 58.6 -> 53.0.  Four waves that move rows into place gain nothing (34.0 -> 36),
// nor does the 64 x 64 tile (1001^3 9.8 -> 11.1): a wave alone on its SIMD pays for the moves what the look-ups give.
// The matrix pipes are busy for 0.25 of the cycles now, the LDS for 0.34.  The line between the two numbers of waves: ragged_layout.h.
#pragma once
#include <type_traits>

#include "ge_device.h"
#include "ragged_layout.h"

namespace ge {

// The chunks of one operand that a lane brings in per 64-k step of a tile BX wide (ragged_layout.h).
// NW: waves of the workgroup; eight read rows at odd elements from 4-byte addresses and move them into place.
template <int BX, bool STRIDED, int NW>
struct RaggedChunks {
    static constexpr int NL = BX / 8 / NW, ROWS = ragged_rows<BX, STRIDED>();
    static constexpr bool MOVE = NW == 8;
    // (ragged_layout.h counts the chunks of four waves)
    __device__ __forceinline__ static constexpr int of_four(int j, int w) { return NW == 8 ? 2 * j + (w >> 2) : j; }
    int off[NL], offLast[NL];               // byte offset of each chunk from the step's first element: in any step but the last, in the last
    int ld, left;                           // leading dimension; rows (columns) of the operand from the tile's first
    bool odd;                               // some row starts at an odd element (wave-uniform)
    unsigned pick;                          // this lane's rows: a dword of them out of two neighbouring ones that were read
    int slot;

    // g: the first step's first element
    __device__ __forceinline__ void init(const char *g, int ld_, int left_, int kLast, int w, int lane)
    {
        ld = ld_;
        left = left_;
        const unsigned base = (unsigned)(uintptr_t)g >> 1;
        odd = MOVE && ((base | (unsigned)ld) & 1u);
        slot = MOVE ? ragged_slot<BX, STRIDED>(w & 3, lane) : lane;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab, sh;
            long long at;
            ragged_place<BX, STRIDED>(of_four(j, w), w & 3, slot, r, c, slab);
            const unsigned o = ragged_offset<STRIDED, 8>(r, c, ld, left);
            off[j] = (int)(o + (MOVE ? (base + o) & 1u : 0u)) * 2;
            ragged_last<STRIDED, 8>(r, c, ld, left, kLast, at, sh);
            offLast[j] = (int)at * 2;
            // (the rows of a lane's chunks are multiples of 16 apart, so all start at odd elements or none does)
            if (j == 0) pick = (base + (unsigned)r * (unsigned)ld) & 1u ? 0x05040302u : 0x07060504u;
        }
    }
    __device__ __forceinline__ void load(const char *step, bool last, i32x4_t (&v)[NL]) const
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) v[j] = ((const i32x4_any_t *)(step + (last ? offLast[j] : off[j])))->v;
    }
    // a step that is not the last: rows read from their second element on move up by one, behind the end of the chunk before
    // (the first chunk of a row gets its first element from elsewhere)
    __device__ __forceinline__ void settle(i32x4_t (&v)[NL]) const
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int before = __builtin_amdgcn_update_dpp(0, v[j][3], 0x111, 0xf, 0xf, true);       // row_shr:1, the lane before
#pragma unroll
            for (int i = 3; i >= 0; --i) v[j][i] = (int)__builtin_amdgcn_perm((unsigned)v[j][i], (unsigned)(i ? v[j][i - 1] : before), pick);
        }
    }
    // what the last step read is put in its place when it has arrived
    __device__ __forceinline__ void settle_last(int kLeft, int w, i32x4_t (&v)[NL]) const
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab, sh;
            long long at;
            ragged_place<BX, STRIDED>(of_four(j, w), w & 3, slot, r, c, slab);
            ragged_last<STRIDED, 8>(r, c, ld, left, kLeft, at, sh);
            v[j] = shift_down_elements(v[j], sh);
        }
    }
    __device__ __forceinline__ void store(GE_LDS char *stage, int w, const i32x4_t (&v)[NL]) const
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab;
            ragged_place<BX, STRIDED>(of_four(j, w), w & 3, slot, r, c, slab);
            *(GE_LDS i32x4_t *)(stage + slab * 1024 + slot * 16) = v[j];
        }
    }
};

// an element of a stage that holds 16-byte chunks
typedef unsigned short __attribute__((may_alias)) u16_alias_t;

// A stored M x K or (TA) K x M, B stored K x N or (TB) N x K.  MODE: 0 fp32 partial sums of one K slice, 1 the run-time
// consumer chain with fp32 output, 2 with bf16 output.  Four waves (NW) in a 2 x 2 or eight in
// a 2 x 4 arrangement on a BT x BT tile.  ONE: a block's K is one step at most (a kernel of its own: as a branch of the other
// it took registers from that, and eight waves spilled).
template <int BT, int NW, bool TA, bool TB, int MODE, bool ONE>
__global__ void __launch_bounds__(NW * 64, NW / 2)
gemm_bf16_ragged_kernel(const GemmParams p)
{
    constexpr int WAVES_N = NW / 2;
    constexpr int WTM = BT / 2, WTN = BT / WAVES_N, TM = WTM / 16, TN = WTN / 16, STAGE = BT * 128, IMAGE32 = BT * 64;
    using ChunksA = RaggedChunks<BT, TA, NW>;
    using ChunksB = RaggedChunks<BT, !TB, NW>;
    // A stages 0 and 1, then B stages 0 and 1
    __shared__ __attribute__((aligned(1024))) char smem[4 * STAGE];
    GE_LDS char *const lds = (GE_LDS char *)smem;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w / WAVES_N, wn = w % WAVES_N;
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
    ca.init(gA, p.lda, p.M - m0, kLast, w, lane);
    cb.init(gB, p.ldb, p.N - n0, kLast, w, lane);
    // First elements of the rows that this wave brings in, A's by the lower half of its lanes and B's by the upper.  Lanes beyond
    // those, and all where no row is odd, read one element that is not stored.
    constexpr int FIRSTS_A = ChunksA::NL * ChunksA::ROWS, FIRSTS_B = ChunksB::NL * ChunksB::ROWS;
    const bool ofA = lane < 32;
    const int first = lane & 31;
    const bool firstOdd = ofA ? ca.odd && first < FIRSTS_A : cb.odd && first < FIRSTS_B;
    int firstAt, firstOff;
    {
        int rA, rB, atA, atB;
        ragged_first<BT, TA>(ChunksA::of_four(first % FIRSTS_A / ChunksA::ROWS, w), first % ChunksA::ROWS, w & 3, rA, atA);
        ragged_first<BT, !TB>(ChunksB::of_four(first % FIRSTS_B / ChunksB::ROWS, w), first % ChunksB::ROWS, w & 3, rB, atB);
        firstAt = ofA ? atA : 2 * STAGE + atB;
        firstOff = !firstOdd ? 0 : ofA ? (int)ragged_offset<TA, 8>(rA, 0, p.lda, p.M - m0) * 2 : (int)ragged_offset<!TB, 8>(rB, 0, p.ldb, p.N - n0) * 2;
    }
    // two register sets: even steps travel in set 0 to LDS stage 0, odd ones in set 1 to stage 1.  Steps beyond the last
    // are the last one again, so that no load sits behind a branch (whose two sides the compiler joins by copying
    // the registers, which waits for the loads).
    i32x4_t va[2][ChunksA::NL], vb[2][ChunksB::NL];
    unsigned short vf[2];
    auto load = [&](int t, auto set) {
        constexpr int S = decltype(set)::value;
        const bool last = t + 1 >= nk;
        const int tt = last ? nk - 1 : t;
        const char *sA = gA + tt * stepA, *sB = gB + tt * stepB;
        ca.load(sA, last, va[S]);
        cb.load(sB, last, vb[S]);
        if constexpr (NW == 8) vf[S] = *(const unsigned short *)((ofA ? sA : sB) + (last ? 0 : firstOff));
    };
    auto store = [&](auto set, bool last) {
        constexpr int S = decltype(set)::value;
        if (last) {
            ca.settle_last(kLast, w, va[S]);
            cb.settle_last(kLast, w, vb[S]);
        } else {
            if (ca.odd) ca.settle(va[S]);
            if (cb.odd) cb.settle(vb[S]);
        }
        ca.store(lds + S * STAGE, w, va[S]);
        cb.store(lds + (2 + S) * STAGE, w, vb[S]);
        if (NW == 8 && !last && firstOdd) *(GE_LDS u16_alias_t *)(lds + S * STAGE + firstAt) = vf[S];       // (after the chunks: a wave's writes to LDS stay in order)
    };
    auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // fragment addresses as in the main kernel: one base per k half of a 128-byte-row stage, one per 16-row block of
    // a k-strided one
    unsigned aAt[TA ? TM : 2], bAt[TB ? 2 : TN];
#pragma unroll
    for (int i = 0; i < (TA ? TM : 2); ++i)
        aAt[i] = TA ? (unsigned)b_frag_offset<BT>(wm * WTM, lane, 0) ^ (unsigned)(i * 32) : (unsigned)a64_frag_offset(wm * WTM, lane, i);
#pragma unroll
    for (int j = 0; j < (TB ? 2 : TN); ++j)
        bAt[j] = (unsigned)(2 * STAGE) + (TB ? (unsigned)a64_frag_offset(wn * WTN, lane, j) : (unsigned)b_frag_offset<BT>(wn * WTN, lane, 0) ^ (unsigned)(j * 32));
    auto read_strided = [&](unsigned at) {
        const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)(lds + at));
        const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)(lds + at + 4 * BT * 2));
        return __builtin_bit_cast(bf16x8_t, (short8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.0f;

    auto multiply = [&](int s) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8_t fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (TA) fa[i] = read_strided(aAt[TA ? i : 0] + (unsigned)(s * STAGE + h * IMAGE32));
                else fa[i] = *(const GE_LDS bf16x8_t *)(lds + aAt[TA ? 0 : h] + s * STAGE + i * 2048);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (TB) fb[j] = *(const GE_LDS bf16x8_t *)(lds + bAt[TB ? h : 0] + s * STAGE + j * 2048);
                else fb[j] = read_strided(bAt[TB ? 0 : j] + (unsigned)(s * STAGE + h * IMAGE32));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
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
    if constexpr (ONE) {                      // nothing to ask for ahead: below, a short K reads its one step three times over
        if (nk > 0) {
            load(0, S0{});
            store(S0{}, true);
            barrier();
            multiply(0);
            barrier();
        }
    } else if (nk > 0) {
        load(0, S0{});
        load(1, S1{});
        store(S0{}, nk == 1);
        load(2, S0{});
        barrier();
        int t = 0;
        for (; t + 3 < nk; t += 2) {          // neither of the two steps written here is the last
            store(S1{}, false);
            load(t + 3, S1{});
            multiply(0);
            barrier();
            store(S0{}, false);
            load(t + 4, S0{});
            multiply(1);
            barrier();
        }
        // one, two or three steps are left, the first of them in stage 0
        const int left = nk - t;
        if (left > 1) store(S1{}, left == 2);
        multiply(0);
        if (left > 1) {
            barrier();
            if (left > 2) store(S0{}, true);
            multiply(1);
            if (left > 2) {
                barrier();
                multiply(0);
            }
        }
        barrier();
    }

    if constexpr (MODE == 2) {
        fused_epilogue_bf16_through_lds<BT, BT, NW, 4 * STAGE, TM, TN, true, false, true>(
            p, tc.b, acc, lds, m0, n0, wm * WTM + (lane & 15), wn * WTN + 4 * (lane >> 4), w, lane);
    } else {
        const int rowLane = m0 + wm * WTM + 4 * (lane >> 4), colLane = n0 + wn * WTN + (lane & 15);
        if constexpr (MODE == 1) {
            if (tile_inside(m0, BT, p.M) && tile_inside(n0, BT, p.N)) fused_epilogue_f32_direct<TM, TN, false>(p, tc.b, acc, rowLane, colLane);
            else fused_epilogue_f32_direct<TM, TN, true>(p, tc.b, acc, rowLane, colLane);
        } else {
            float *cBase = p.C + (long long)tc.s * p.sliceStride + (long long)tc.b * p.M * p.N;
            if (tile_inside(m0, BT, p.M) && tile_inside(n0, BT, p.N)) store_plain_tile<true, ACT_NONE, false>(nullptr, 1.0f, cBase, p.N, p.M, p.N, acc, rowLane, colLane);
            else store_plain_tile<true, ACT_NONE, true>(nullptr, 1.0f, cBase, p.N, p.M, p.N, acc, rowLane, colLane);
        }
    }
}

}  // namespace ge
