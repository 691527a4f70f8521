// gemm_bf16_ragged_kernel on 128 x 128 tiles: the choice between four and eight waves, and every operand storage and output mode
// with four.
#include "gemm_ragged_tiles.h"

namespace ge_host {

// Eight waves where a block has its CU to itself, or where both operands have rows at odd elements: more blocks cover each other's
// waits, and then only the look-ups saved count.  us, four / eight waves: 208 blocks, 1999 x 1537 x 2051 33.8 / 31.5, aligned rows
// 27.9 / 27.5, A stored K x M 1999 x 1537 x 515 14.8 / 12.7; more blocks, both odd, 2047 x 2049 x 2051 53.8 / 49.0, 3001 x 3001 x 901
// 41.9 / 40.5, 4095 x 4093 x 2047 108.4 / 104.3; one odd, 4001 x 3003 x 700 33.8 / 34.5, 3000 x 3001 x 1024 40.7 / 41.4; none, 2500 x
// 3001 x 704 with B stored N x K 19.3 / 19.7.  Not with both odd where odd leading dimensions make every other row so, B is stored N x K and
// there are four blocks to a CU: half of what is moved was in place (201 x 3520 x 1433, 20 of them, 102.6 / 115.8; 1724 x 1680 x 77, 20,
// 70.8 / 81.2; fewer blocks 2047 x 2049 x 2051, 52.0 / 47.5).  One step of K is never moved: four waves, in the kernel that asks for no more, but for
// few blocks (4001 x 3003 x 60 with A stored K x M, 768 blocks, 12.3 / 16.2; 1341 x 104 x 48, 20 of them, 220 blocks, 7.5 / 6.9).
void launch_ragged_128(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st)
{
    if (p.kPerSlice <= 64 && grid.x > (unsigned)kNumCU) return launch_ragged_tile<128, 4, true>(p, raw, grid, st);
    const bool oddA = (p.lda & 1) || ((uintptr_t)p.A & 2u), oddB = (p.ldb & 1) || ((uintptr_t)p.B & 2u);
    const bool half = (p.lda & 1) && (p.ldb & 1) && p.transB && grid.x >= 4u * kNumCU;
    if (grid.x <= (unsigned)kNumCU || (oddA && oddB && !half)) launch_ragged_128_w8(p, raw, grid, st);
    else launch_ragged_tile<128, 4, false>(p, raw, grid, st);
}

}  // namespace ge_host
