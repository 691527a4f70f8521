// gemm_bf16_ragged_kernel on 128 x 128 tiles: the choice between four and eight waves (ragged_layout.h), and every operand storage and output
// mode with four.
#include "gemm_ragged_tiles.h"

namespace ge_host {

void launch_ragged_128(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st)
{
    static_assert(ge::RAGGED_CUS == kNumCU, "the line between the numbers of waves counts CUs");
    const bool oddA = (p.lda & 1) || ((uintptr_t)p.A & 2u), oddB = (p.ldb & 1) || ((uintptr_t)p.B & 2u);
    const double m = p.M, n = p.N, k = p.K, bytes = p.batch * (2.0 * (m + n) * k + (raw ? 4.0 * p.splitK : p.cType == ge::DT_BF16 ? 2.0 : 4.0) * m * n);
    const ge::RaggedWaves w = ge::ragged_128_waves(grid.x, p.kPerSlice, oddA, oddB, (p.lda & 1) && (p.ldb & 1), p.transA, p.transB, bytes);
    if (w.waves == 8) launch_ragged_128_w8(p, raw, grid, st);
    else if (w.one)   launch_ragged_tile<128, 4, true>(p, raw, grid, st);
    else              launch_ragged_tile<128, 4, false>(p, raw, grid, st);
}

}  // namespace ge_host
