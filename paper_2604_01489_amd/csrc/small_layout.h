// Which 16-byte chunk of an operand each lane brings in, and where it lies in LDS, for the kernel of few output tiles (gemm_small.h), as
// plain index functions that are compiled into the kernel and into the host-side model test.  The images are bf16_layout.h's, four of 64 k to a step.
#pragma once
#include "bf16_layout.h"
#include "ragged_layout.h"

namespace ge {

constexpr int SMALL_STEP = 256;             // k of a step

// Chunks that a lane of NW waves brings in per step of an operand BX wide
template <int BX, int NW>
GE_HD constexpr int small_chunks() { return BX / 2 / NW; }

// Chunk j of a lane of wave w: its row (k row of the step if STRIDED) and chunk along it (of the step if not), and its place in the operand's
// stage; neighbouring lanes, neighbouring chunks of a row, a wave's chunks within one image of 64 k.
template <int BX, int NW, bool STRIDED>
GE_HD constexpr void small_place(int j, int w, int lane, int &r, int &c, int &at)
{
    constexpr int PER_IMAGE = BX / 8;                        // wave-wide loads
    const int idx = w * small_chunks<BX, NW>() + j, image = idx / PER_IMAGE, q = (idx % PER_IMAGE) * 64 + lane;
    if constexpr (STRIDED) {
        const int k = q / (BX / 8);
        c = q % (BX / 8);
        r = image * 64 + k;
        at = image * (BX * 128) + (k / 32) * (BX * 64) + lds_b_offset<BX>(k % 32, c);
    } else {
        r = q / 8;
        c = image * 8 + q % 8;
        at = image * (BX * 128) + lds_a64_offset(r, q % 8);
    }
}

// Whether rows at odd elements make fp32 results of any alignment and 257 to 320 k, the first of a second step of 256, the slower ones in 32 x 32 tiles: every chunk of them costs
// twice the look-ups, and the second step brings in as many as the first.  1800 drawn calls, of the time on the 64 x 64 tile with and without such rows: without a residual, A stored K x M odd 1.03 to
// 1.07, else 0.95 to 0.99, M x K with both odd 1.03, else 0.95 to 1.00 (199 x 465 x 273, A K x M, B N x K, 5.3 / 5.8; 277 x 842 x 269 5.3 / 5.7; 38 x 618 x 320 5.35 / 4.9); with one, A K x M with both odd 1.02 and
// 1.00, else 0.94 to 0.99.  (bf16 out 0.95 to 1.00, in one call of thirty above 1.03, to 1.08.)
GE_HD constexpr bool small_odd_rows(bool transA, bool oddA, bool oddB, bool residual) { return transA ? oddA && (oddB || !residual) : oddA && oddB && !residual; }

// Whether a product whose plan names the 128 x 128 tile or (ragged) the 64 x 64 one of gemm_ragged.h goes to workgroups in 32 x 32 tiles: tiles of those,
// K slices of the plan, K; oddRows: fp32 out with rows as above.  Up to one tile to a CU it does: us, plan's tile / small, 192 x 312 x 640 6.5 / 5.0, 264 x 232 x 1920 12.5 / 8.6 (B N x K,
// bf16 out, 11.9 / 7.7), 72 x 1096 x 1160 9.0 / 6.2, 200^3 5.8 / 3.7, 512^3 5.8 / 4.9; over 21000 drawn calls 0.72 of the time on average.  Not where the 64 x 64 tile has
// one 64-k step, for which it has a kernel of its own (533 x 416 x 47 3.6 / 4.0).
// Beyond that only what is over in one step of 256, which has no walk to wait in: more than 128 k, up to two tiles a CU beside the 64 x 64 tile
// (0.83 to 0.98 of its time) or three beside the 128 x 128 one (0.7 to 0.98; four 1.1); more than 64 k, two beside the latter (0.8 to 0.94; K <= 64 1.02; 640^3, 400 tiles, 6.5 / 6.9).
// In place of K slices, which cost a second launch and its round trip, where one walk over K is the shorter way: 512 x 512 x 2048, four slices, 10.9 / 8.9, 44 x 690 x
// 1109 8.8 / 6.3; aligned operands, whose slices are the longer kernel's, up to four of them (1900 drawn calls of 2496 to 2552 k 0.79 to 0.87, A K x M in one of a hundred 1.03 to 1.09), and five where
// their second pass has much to add up (26000 drawn calls of 2560 k: A M x K up to 64 tiles 1.00 to 1.06, then 0.86 to 0.97; A K x M up to 192 0.97 to 1.05 with single ones 1.2, then 0.94 to 0.95; 24 x 24 8.9 / 9.6, 280 x
// 168 with A K x M 10.8 / 12.4, 128 x 1464 12.5 / 10.3); the others up to 1536 (36 x 71 x 1653 8.5 / 9.5; 40 x 1678 x 2119 9.1 / 10.9).
constexpr int SMALL_CUS = 256;
GE_HD constexpr bool small_tile_takes(long long tiles, int slices, int K, bool ragged, bool transA, bool oddRows)
{
    if (slices > 1) return tiles <= SMALL_CUS && (ragged ? K <= 1536 : K < 2560 || (K == 2560 && tiles > (transA ? 192 : 64)));
    if (ragged && (K <= 64 || (oddRows && K > SMALL_STEP && K <= 320))) return false;
    if (tiles <= SMALL_CUS) return true;
    if (K > SMALL_STEP || K <= 64) return false;
    return K > 128 ? tiles <= (ragged ? 2 : 3) * SMALL_CUS : !ragged && tiles <= 2 * SMALL_CUS;
}

// The same for a convolution whose plan names the 128 x 128 tile; c8: of the kernel for channels a multiple of 8 but not of 32.  That tile's gathered
// steps take 0.2 to 0.35 us each beside 8 us for its prologue and epilogue, more than in a product, so the lines lie further out.  us, plan's tile / small: 8 images of 14 x 14 x 256 -> 64, 1 x 1, 6.9 / 3.9; 14 of 13 x 13 x 256 -> 32, 3 x 3, in slices 11.9 / 9.4; of its time over 9000 drawn
// calls, up to two tiles a CU: K = 64 0.78 to 0.91, 256 0.55 to 0.65, 576 0.56 to 0.70, 1152 0.46 to 0.58, in slices 2304 0.72 to 0.86 (4608 1.0 to 1.4), c8 0.38 to 0.9.  Three: 65 to 256 k 0.94
// and 0.77, 1152 0.87, c8 0.70 to 0.85 (288 to 576 k 1.0 to 1.24); four: 129 to 256 k 0.87.  These with bf16 out; fp32 out without a residual (bareF32), whose stores are
// twice as many, beside the larger tile's in one round of them: a second tile a CU from 48 k on (48 0.97, 64 1.00; 32 1.05: 3724 x 128 x 32 4.7 / 5.1; 16 1.03), a third from 129 on
// (128 1.04: 6125 x 128 x 128 5.8 / 6.1; channels of 8, 80 k, 1.05), as with bf16 out beyond that; what stays takes the 64 x 128 tile (0.84 to 0.87).  With a residual as with bf16 out (32 k 0.90, 128 0.91).
GE_HD constexpr bool small_conv_takes(long long tiles, int slices, int K, bool c8, bool bareF32)
{
    if (slices > 1) return tiles <= 2 * SMALL_CUS && K <= 2560;
    if (bareF32 && tiles > SMALL_CUS && K <= (tiles > 2 * SMALL_CUS ? 128 : 47)) return false;
    if (tiles <= 2 * SMALL_CUS) return true;
    if (K > 128 && K <= SMALL_STEP) return tiles <= 4 * SMALL_CUS;
    return tiles <= 3 * SMALL_CUS && (K <= 128 ? K > 64 : K > 768 || c8);
}

// Which of the tiles of gemm_tile64_launch.h (figures there) a product in one pass takes whose plan names the 128 x 128 tile (plan128) or the 256 x 256 one; blocks: its 64 x 128 tiles;
// oddRows: their rows are odd in number; upTo: the K up to which it takes the 64 x 128 tile beyond one block a CU.
enum Tile64 { TILE64_NO = 0, TILE64_RING = 1, TILE64_SHORT = 2, TILE64_SHORT_WIDE = 3 };
GE_HD constexpr Tile64 tile64_kind(bool plan128, long long blocks, int K, bool bf16Out, bool oddRows, int upTo = 128)
{
    // three are on a CU at once, or two of 128 x 128: what four to a CU take twice, those take in one round
    const bool third = blocks <= 3 * SMALL_CUS, fourth = !third && blocks <= 4 * SMALL_CUS;
    if (K > 64) {
        if (plan128 && blocks <= SMALL_CUS) return TILE64_RING;
        return bf16Out && K <= upTo && (plan128 ? !fourth && blocks <= 6 * SMALL_CUS : !third && blocks <= 5 * SMALL_CUS) ? TILE64_RING : TILE64_NO;
    }
    if (bf16Out) return fourth || blocks > 16 * SMALL_CUS ? TILE64_SHORT_WIDE : TILE64_SHORT;
    return plan128 && (blocks <= SMALL_CUS || (blocks > 4 * SMALL_CUS && blocks <= (oddRows ? 16 : 5) * SMALL_CUS)) ? TILE64_SHORT : TILE64_NO;
}

// A convolution's: with a chunk's tap per lane (c8) the larger tile's steps are dearer.
GE_HD constexpr Tile64 conv_tile64_kind(bool plan128, long long blocks, int K, bool bf16Out, bool oddRows, bool c8)
{
    return tile64_kind(plan128, blocks, K, bf16Out, oddRows, !c8 ? 128 : 2 * blocks <= 3 * SMALL_CUS ? 1152 : blocks <= 2 * SMALL_CUS ? 576 : 256);
}

// Steps whose sums form one chain before they are added to the others: a plan's K slice, so that the sums are as exact as in slices.
GE_HD constexpr int small_run(int slices, int kPerSlice) { return slices > 1 ? (kPerSlice >= SMALL_STEP ? kPerSlice / SMALL_STEP : 1) : 0x7fffffff; }

// fp32 (gemm_f32_few.h): 32 x 32 tiles in steps of 128 k, 16 x 16 ones in steps of 256, 16 KB of either operand to a step.  Rows of A along k and k rows
// of B, padded by 16 bytes: a wave reads 16 bytes of 16 rows of A, and a column's element of k rows four apart of B.
GE_HD constexpr int few_step_f32(int BT) { return 4096 / BT; }
GE_HD constexpr int few_pitch_a(int BT) { return few_step_f32(BT) * 4 + 16; }
GE_HD constexpr int few_pitch_b(int BT) { return BT * 4 + 16; }
GE_HD constexpr int few_at_a(int BT, int row, int k) { return row * few_pitch_a(BT) + k * 4; }
GE_HD constexpr int few_at_b(int BT, int k, int col) { return k * few_pitch_b(BT) + col * 4; }

// chunk j (of four floats) of a lane of wave w: its row (k row if STRIDED), chunk along it, and place in the operand's stage
template <int BT, bool STRIDED>
GE_HD constexpr void few_place_f32(int j, int w, int lane, int &r, int &c, int &at)
{
    constexpr int PER_ROW = (STRIDED ? BT : few_step_f32(BT)) / 4;
    const int q = (j * 4 + w) * 64 + lane;
    r = q / PER_ROW;
    c = q % PER_ROW;
    at = STRIDED ? few_at_b(BT, r, c * 4) : few_at_a(BT, r, c * 4);
}

// The tile an fp32 product of tiles16 16 x 16 tiles, or tiles32 32 x 32 ones, that takes no K slices is dealt out in, or 0: neither, it stays on the larger ones.
// us, 64 x 64 tile / 32 / 16: 256^3 (on tiles of 32 that read from memory directly) 6.2 / 5.5 / 3.8; 142 x 343 x 983 23.2 / 11.6 / 7.2; 80 x 100 x 512 13.0 / 7.7 / 4.9; 320 x 336 x 888
// 21.0 / 11.1 / 9.1; 256 x 938 x 347 10.3 / 7.1 / 10.8; 512^3 8.7 / 8.1 / 11.2; 550 x 192 x 128 5.6 / 4.1 / 4.3; 320 x 1864 x 384, 590 tiles of 32, 11.2 / 13.6 / 22.4.
// 14000 drawn calls: 16 up to two a CU 0.30 (K = 1000) to 0.75 of the time (K = 100), of which the second tile of a CU pays from 128 k on; 32 up to one a CU 0.5 to 0.8, and
// 0.97 for K <= 64; up to two 0.75 to 0.88 with more than 256 k, with fewer 0.9 to 1.1.
GE_HD constexpr int few_tile_f32(long long tiles16, long long tiles32, int K)
{
    if (K > 64 && tiles16 <= (K > 128 ? 2 : 1) * SMALL_CUS) return 16;
    return tiles32 <= (K > 256 ? 2 : 1) * SMALL_CUS ? 32 : 0;
}

}  // namespace ge
