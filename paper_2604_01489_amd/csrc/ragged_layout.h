// Which 16-byte chunk of an operand of any alignment each lane brings in (gemm_ragged.h: bf16, gemm_f32_ragged.h: fp32), as
// plain index functions that are compiled into the kernels and into the host-side model test.  The LDS layouts are
// bf16_layout.h's.  E: elements of a 16-byte chunk, 8 or 4.
//
// bf16: a 64-k step of a tile BX wide is BX * 128 bytes, BX / 32 chunks of 8 elements per lane of the four waves.  STRIDED: the
// operand's memory rows run along the tile's rows (M or N), and a step is two images of 32 k; else they run along k, and
// a step is one image of 128-byte rows.  Offsets are in elements from the step's first one.
#pragma once
#include "bf16_layout.h"

namespace ge {

// chunk j of a lane: its row (k row if STRIDED) and chunk along it, and the 1 KB slab of LDS that it lands in (at 16 * lane)
template <int BX, bool STRIDED>
GE_HD constexpr void ragged_place(int j, int w, int lane, int &r, int &c, int &slab)
{
    if constexpr (STRIDED) {
        constexpr int PER = BX / 64;
        const int h = j / PER, wl = (j % PER) * 4 + w;
        r = 32 * h + b_slot_k<BX>(wl, lane);
        c = b_slot_chunk<BX>(wl, lane);
        slab = h * (BX / 16) + wl;
    } else {
        slab = j * 4 + w;
        r = a64_slot_row(slab, lane);
        c = a64_slot_chunk(slab, lane);
    }
}

// The place in its slab, 16 bytes each, that a lane fills so that neighbouring lanes hold neighbouring chunks of a row (ragged_place
// of that place gives the lane's row and chunk); the same for every j.
template <int BX, bool STRIDED>
GE_HD constexpr int ragged_slot(int w, int lane)
{
    if constexpr (STRIDED) {
        constexpr int PER_ROW = BX / 8;
        return (lane & ~(PER_ROW - 1)) | (lds_b_offset<BX>(b_slot_k<BX>(w, lane) & 31, lane & (PER_ROW - 1)) % (BX * 2) / 16);
    } else {
        return (lane & ~7) | (a64_slot_chunk(w, lane) & 7);
    }
}

// Rows that start at an odd element are read from the element after, at 4-byte addresses, and put together from
// two neighbouring chunks; what then is missing is the first element of each row.  Row i of those that chunk j of a wave's lanes
// covers, and where its first element lies in the stage.
template <int BX, bool STRIDED>
GE_HD constexpr int ragged_rows() { return STRIDED ? 512 / BX : 8; }
template <int BX, bool STRIDED>
GE_HD constexpr void ragged_first(int j, int i, int w, int &r, int &at)
{
    int c = 0, slab = 0;
    ragged_place<BX, STRIDED>(j, w, i * (64 / ragged_rows<BX, STRIDED>()), r, c, slab);
    at = STRIDED ? (r / 32) * (BX * 64) + lds_b_offset<BX>(r % 32, 0) : lds_a64_offset(r, 0);
}

// Waves of a workgroup of the bf16 kernel's 128 x 128 tile, for `blocks` of them, and whether their K is read as one step (`one`: kPerSlice is
// 64 or less).  oddA, oddB: that operand has rows at odd elements; ldsOdd: both leading dimensions are odd, so that every other row is in
// place as it is; bytes: operands and result.
// Eight waves where a block has its CU to itself, or where both operands have rows at odd elements: more blocks cover each other's
// waits, and then only the look-ups saved count.  us, four / eight waves: 208 blocks, 1999 x 1537 x 2051 33.8 / 31.5, aligned rows
// 27.9 / 27.5, A stored K x M 1999 x 1537 x 515 14.8 / 12.7; more blocks, both odd, 2047 x 2049 x 2051 53.8 / 49.0, 3001 x 3001 x 901
// 41.9 / 40.5, 4095 x 4093 x 2047 108.4 / 104.3; one odd, 4001 x 3003 x 700 33.8 / 34.5, 3000 x 3001 x 1024 40.7 / 41.4; none, 2500 x
// 3001 x 704 with B stored N x K 19.3 / 19.7.  Where every other row is in place only half of what is moved gains, and four waves stay:
// - past the 256 MB memory-side cache, where memory and not the look-ups is the bound (112 x 4927 x 4757, 7 of them, B N x K, 164.6 / 196.4;
//   120 x 1770 x 3836, 20, 123.0 / 145.1; 124 x 1300 x 1120, 100, 114.2 / 128.9);
// - B stored N x K with four blocks to a CU (201 x 3520 x 1433, 20, 102.6 / 115.8; 1724 x 1680 x 77, 20, 70.8 / 81.2) or, A M x K, with more than
//   1536 k to a block (1123 x 4209 x 1711 46.8 / 51.1, 1408 x 184 x 1812, 20, 51.0 / 56.2; fewer of both 2047 x 2049 x 515 19.6 / 18.1);
// - three steps of K with A stored K x M and B K x N (1658 x 2678 x 177 11.5 / 12.8, 5373 x 1299 x 191 13.4 / 14.4; two steps 1.00, four 0.97 of it).
// One step of K is never moved: four waves, in the kernel that asks for no more, but for
// few blocks (4001 x 3003 x 60 with A stored K x M, 768 blocks, 12.3 / 16.2; 1341 x 104 x 48, 20 of them, 220 blocks, 7.5 / 6.9).
constexpr int RAGGED_CUS = 256;
struct RaggedWaves { int waves; bool one; };
constexpr RaggedWaves ragged_128_waves(unsigned blocks, int kPerSlice, bool oddA, bool oddB, bool ldsOdd, bool transA, bool transB, double bytes)
{
    if (blocks <= (unsigned)RAGGED_CUS) return {8, false};
    if (kPerSlice <= 64) return {4, true};
    if (!oddA || !oddB) return {4, false};
    const bool four = bytes > 256.0 * 1024 * 1024 || (transB && (blocks >= 4u * RAGGED_CUS || (!transA && kPerSlice > 1536))) ||
                      (transA && !transB && kPerSlice == 192);
    return {ldsOdd && four ? 4 : 8, false};
}

// fp32: a 32-k step of a tile BX wide, BX / 32 chunks per lane, is two images of 16 k: 64-byte rows of A (along k), B in
// rows of BX floats.
template <int BX, bool STRIDED>
GE_HD constexpr void ragged_place_f32(int j, int w, int lane, int &r, int &c, int &slab)
{
    constexpr int PER = BX / 64;
    const int h = j / PER, wl = (j % PER) * 4 + w;
    r = STRIDED ? 16 * h + b_slot_k<2 * BX>(wl, lane) : a_slot_row(wl, lane);
    c = STRIDED ? b_slot_chunk<2 * BX>(wl, lane) : 4 * h + a_slot_chunk(lane);
    slab = h * (BX / 16) + wl;
}

// A step that is not the block's last: `left` is the number of the operand's rows (columns if STRIDED) from the tile's
// first.  Rows beyond are the last one again, chunks beyond the end of a row along M or N the tile's first; a chunk that
// hangs over such an end reads on into the row after it, which exists: the step is not the last, and the rows (hence the
// leading dimension) are at least E elements long.  One that is read an element further on, as rows at odd elements are,
// ends inside the next step or the row after it as well.
template <bool STRIDED, int E>
GE_HD constexpr unsigned ragged_offset(int r, int c, int ld, int left)
{
    return STRIDED ? (unsigned)r * (unsigned)ld + (c * E < left ? (unsigned)(c * E) : 0u)
                   : (unsigned)(r < left ? r : left - 1) * (unsigned)ld + (unsigned)(c * E);
}

// The last step, kLeft (at least 1) k of it inside: the chunk is pulled back until it ends inside its row, and what was read
// is shifted down by sh elements (E or more: nothing of it is wanted), which puts zeros beyond the end.
template <bool STRIDED, int E>
GE_HD constexpr void ragged_last(int r, int c, int ld, int left, int kLeft, long long &off, int &sh)
{
    if constexpr (STRIDED) {
        const int start = c * E < left ? c * E : 0, avail = left - start, back = avail < E ? E - avail : 0;
        off = (long long)(r < kLeft ? r : kLeft - 1) * ld + start - back;
        sh = r < kLeft ? back : E;
    } else {
        const int first = c * E <= kLeft - E ? c * E : kLeft - E;
        off = (long long)(r < left ? r : left - 1) * ld + first;
        sh = c * E - first;
    }
}

}  // namespace ge
