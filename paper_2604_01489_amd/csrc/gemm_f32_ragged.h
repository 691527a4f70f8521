// fp32 GEMM for operands the direct-to-LDS kernel does not take (gemm_f32_fast.h): rows that start at any 4-byte address,
// sizes and leading dimensions that are multiples of nothing.  The same matrix instructions (v_mfma_f32_32x32x2_f32), LDS
// layouts and fragment reads; the tile comes through registers, 16 bytes a lane at whatever address, and only the last
// K step of a block guards its reads (ragged_layout.h).
//
// What bounds it: the fp32 matrix pipe where the tiles fill the chip (a 16-k step of a 64 x 64 tile is 512 cycles of it,
// for 16 KB of LDS traffic), and how long a block waits for memory where they do not: two steps of loads are on their way
// in registers while a third is multiplied.
#pragma once
#include <type_traits>

#include "ge_device.h"
#include "ragged_layout.h"

namespace ge {

struct __attribute__((packed, aligned(4))) f32x4_any_t { f32x4_t v; };

// ELEMENTWISE: every element is fetched under its own test (rows shorter than a chunk, panels or a C
// beyond 31-bit offsets).
template <int BX, bool STRIDED, bool ELEMENTWISE>
struct RaggedChunksF32 {
    static constexpr int NL = BX / 32;
    int off[NL], offLast[NL];               // byte offset of each chunk from the step's first element: in any step, in the last
    int ld, left, kLast;                    // leading dimension; rows (columns) of the operand from the tile's first; k of the last step

    __device__ __forceinline__ void init(int ld_, int left_, int kLast_, int w, int lane)
    {
        ld = ld_;
        left = left_;
        kLast = kLast_;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab, sh;
            long long at;
            ragged_place_f32<BX, STRIDED>(j, w, lane, r, c, slab);
            off[j] = (int)ragged_offset<STRIDED, 4>(r, c, ld, left) * 4;
            ragged_last<STRIDED, 4>(r, c, ld, left, kLast, at, sh);
            offLast[j] = (int)at * 4;
        }
    }
    __device__ __forceinline__ void load(const char *step, bool last, int w, int lane, f32x4_t (&v)[NL]) const
    {
        if constexpr (ELEMENTWISE) {
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                int r, c, slab;
                ragged_place_f32<BX, STRIDED>(j, w, lane, r, c, slab);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = STRIDED ? r : c * 4 + e, x = STRIDED ? c * 4 + e : r;
                    v[j][e] = (!last || k < kLast) && x < left ? ((const float *)step)[STRIDED ? (long long)k * ld + x : (long long)x * ld + k] : 0.0f;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < NL; ++j) v[j] = ((const f32x4_any_t *)(step + (last ? offLast[j] : off[j])))->v;
        }
    }
    // what the last step read is put in its place when it has arrived
    __device__ __forceinline__ void settle_last(int w, int lane, f32x4_t (&v)[NL]) const
    {
        if constexpr (ELEMENTWISE) return;
        const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab, sh;
            long long at;
            ragged_place_f32<BX, STRIDED>(j, w, lane, r, c, slab);
            ragged_last<STRIDED, 4>(r, c, ld, left, kLast, at, sh);
            f32x4_t t = v[j];
            t = sh & 1 ? __builtin_shufflevector(t, zero, 1, 2, 3, 4) : t;
            t = sh & 2 ? __builtin_shufflevector(t, zero, 2, 3, 4, 4) : t;
            v[j] = sh >= 4 ? zero : t;
        }
    }
    __device__ __forceinline__ static void store(GE_LDS char *stage, int w, int lane, const f32x4_t (&v)[NL])
    {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int r, c, slab;
            ragged_place_f32<BX, STRIDED>(j, w, lane, r, c, slab);
            *(GE_LDS f32x4_t *)(stage + slab * 1024 + lane * 16) = v[j];
        }
    }
};

// Four waves in a 2 x 2 arrangement on a BT x BT tile, K step 32.  RAW: fp32 partial sums of one K slice.
template <int BT, bool RAW, bool ELEMENTWISE>
__global__ void __launch_bounds__(256, 2)
gemm_f32_ragged_kernel(const GemmParams p)
{
    constexpr int T = BT / 64, WT = BT / 2, IMAGE16 = BT * 64, STAGE = 2 * IMAGE16;
    using ChunksA = RaggedChunksF32<BT, false, ELEMENTWISE>;
    using ChunksB = RaggedChunksF32<BT, true, ELEMENTWISE>;
    // A stages 0 and 1, then B stages 0 and 1
    __shared__ __attribute__((aligned(1024))) char smem[4 * STAGE];
    GE_LDS char *const lds = (GE_LDS char *)smem;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w >> 1, wn = w & 1;
    const TileCoord tc = map_block(p);
    const int m0 = tc.tm * BT, n0 = tc.tn * BT;
    const int kBegin = tc.s * p.kPerSlice, kLen = min(p.K, kBegin + p.kPerSlice) - kBegin;
    const int nk = (kLen + 31) / 32, kLast = kLen - (nk - 1) * 32;      // steps; k of the last one

    const char *gA = (const char *)p.A + 4 * ((long long)tc.b * p.strideA + (long long)m0 * p.lda + kBegin);
    const char *gB = (const char *)p.B + 4 * ((long long)tc.b * p.strideB + (long long)kBegin * p.ldb + n0);
    const long long stepB = (long long)p.ldb * 128;
    ChunksA ca;
    ChunksB cb;
    ca.init(p.lda, p.M - m0, kLast, w, lane);
    cb.init(p.ldb, p.N - n0, kLast, w, lane);
    // two register sets: even steps travel in set 0 to LDS stage 0, odd ones in set 1 to stage 1; steps beyond the last are
    // the last one again, so that no load sits behind a branch
    f32x4_t va[2][ChunksA::NL], vb[2][ChunksB::NL];
    auto load = [&](int t, auto set) {
        constexpr int S = decltype(set)::value;
        const bool last = t + 1 >= nk;
        const int tt = last ? nk - 1 : t;
        ca.load(gA + tt * 128ll, last, w, lane, va[S]);
        cb.load(gB + tt * stepB, last, w, lane, vb[S]);
    };
    auto store = [&](auto set) {
        constexpr int S = decltype(set)::value;
        ChunksA::store(lds + S * STAGE, w, lane, va[S]);
        ChunksB::store(lds + (2 + S) * STAGE, w, lane, vb[S]);
    };
    auto settle = [&](auto set) {
        constexpr int S = decltype(set)::value;
        ca.settle_last(w, lane, va[S]);
        cb.settle_last(w, lane, vb[S]);
    };
    auto barrier = [&] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // fragments as in the direct-to-LDS kernel: A (i, rho): row 32 i + lane%32, chunk 2 rho + lane/32; B (j, rho, e):
    // k = 8 rho + 4 (lane/32) + e, column 32 j + lane%32
    const int g = lane >> 5, l32 = lane & 31;
    unsigned aAt[2], bAt[T][2][4];
#pragma unroll
    for (int rho = 0; rho < 2; ++rho) aAt[rho] = (unsigned)lds_a_offset(wm * WT + l32, 2 * rho + g);
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
        for (int rho = 0; rho < 2; ++rho)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int n = wn * WT + 32 * j + l32;
                bAt[j][rho][e] = (unsigned)(2 * STAGE + lds_b_offset<2 * BT>(8 * rho + 4 * g + e, n >> 2) + (n & 3) * 4);
            }

    f32x16_t acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    auto multiply = [&](auto set) {
        constexpr int S = decltype(set)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int rho = 0; rho < 2; ++rho) {
                f32x4_t a[T];
                float b[T][4];
#pragma unroll
                for (int i = 0; i < T; ++i) a[i] = *(const GE_LDS f32x4_t *)(lds + aAt[rho] + S * STAGE + h * IMAGE16 + i * 2048);
#pragma unroll
                for (int j = 0; j < T; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[j][e] = *(const GE_LDS float *)(lds + bAt[j][rho][e] + S * STAGE + h * IMAGE16);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
            }
    };

    // One barrier per step: step t writes the stage that step t - 1 read, from registers that were asked for two steps
    // ago, and asks memory for step t + 3.  (A block has at least one step: K >= 1, slices are not empty.)
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    load(0, S0{});
    load(1, S1{});
    if (nk == 1) settle(S0{});
    store(S0{});
    load(2, S0{});
    barrier();
    int t = 0;
    for (; t + 3 < nk; t += 2) {              // neither of the two steps written here is the last
        store(S1{});
        load(t + 3, S1{});
        multiply(S0{});
        barrier();
        store(S0{});
        load(t + 4, S0{});
        multiply(S1{});
        barrier();
    }
    // one, two or three steps are left, the first of them in stage 0
    const int rest = nk - t;
    if (rest > 1) {
        if (rest == 2) settle(S1{});
        store(S1{});
    }
    multiply(S0{});
    if (rest > 1) {
        barrier();
        if (rest > 2) {
            settle(S0{});
            store(S0{});
        }
        multiply(S1{});
        if (rest > 2) {
            barrier();
            multiply(S0{});
        }
    }

    // accumulator register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32
    const int rowLane = m0 + wm * WT + 4 * g, colLane = n0 + wn * WT + l32;
    float *cBase = p.C + (long long)tc.b * p.strideC + (RAW ? (long long)tc.s * p.sliceStride : 0ll);
    auto store_tile = [&](auto masked, auto actC) {
        constexpr bool MASK = decltype(masked)::value;
        constexpr int ACT = decltype(actC)::value;
        float bv[T];
        unsigned at[T];
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int n = !MASK || colLane + j * 32 < p.N ? colLane + j * 32 : p.N - 1;
            bv[j] = !RAW && p.bias != nullptr ? p.bias[n] : 0.0f;
            if (MASK && !ELEMENTWISE) at[j] = edge_offset(4 * g, l32 + 32 * j, p.ldc, colLane - l32, p.N);
        }
#pragma unroll
        for (int i = 0; i < T; ++i) {
            buffer_t rows;
            if constexpr (MASK && !ELEMENTWISE) rows = edge_rows<32>(cBase, p.ldc, m0 + wm * WT + i * 32, p.M, colLane - l32, p.N);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int inBlock = 8 * (r >> 2) + (r & 3), m = rowLane + i * 32 + inBlock;
                float v[T];
#pragma unroll
                for (int j = 0; j < T; ++j) v[j] = acc[i][j][r];
                if (!RAW) epilogue_values<ACT, T>(v, p.alpha, bv);
#pragma unroll
                for (int j = 0; j < T; ++j) {
                    if constexpr (MASK && !ELEMENTWISE) edge_store(rows, at[j], inBlock, p.ldc, v[j]);
                    else if (!MASK || (m < p.M && colLane + j * 32 < p.N)) cBase[(long long)m * p.ldc + colLane + j * 32] = v[j];
                }
            }
        }
    };
    // the case of the activation, then the mask of a tile on the edge: uniform branches around the whole tile
    auto store_by_mask = [&](auto actC) {
        if (tile_inside(m0, BT, p.M) && tile_inside(n0, BT, p.N)) store_tile(std::false_type{}, actC);
        else store_tile(std::true_type{}, actC);
    };
    if (RAW || p.act == ACT_NONE) store_by_mask(std::integral_constant<int, ACT_NONE>{});
    else if (p.act == ACT_RELU) store_by_mask(std::integral_constant<int, ACT_RELU>{});
    else store_by_mask(std::integral_constant<int, ACT_GELU_TANH>{});
}

}  // namespace ge
