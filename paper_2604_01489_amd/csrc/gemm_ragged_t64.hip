// gemm_bf16_ragged_kernel on 64 x 64 tiles: every operand storage and output mode.
#include "gemm_ragged_tiles.h"

namespace ge_host {

void launch_ragged_64(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st)
{
    if (p.kPerSlice <= 64) launch_ragged_tile<64, 4, true>(p, raw, grid, st);
    else                   launch_ragged_tile<64, 4, false>(p, raw, grid, st);
}

}  // namespace ge_host
