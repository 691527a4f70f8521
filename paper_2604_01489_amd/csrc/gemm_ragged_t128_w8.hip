// gemm_bf16_ragged_kernel on 128 x 128 tiles with eight waves to a workgroup: every operand storage and output mode.
#include "gemm_ragged_tiles.h"

namespace ge_host {

void launch_ragged_128_w8(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st) { launch_ragged_tile<128, 8, false>(p, raw, grid, st); }

}  // namespace ge_host
