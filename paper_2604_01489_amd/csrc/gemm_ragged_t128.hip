// gemm_bf16_ragged_kernel on 128 x 128 tiles: every operand storage and output mode.
#include "gemm_ragged_tiles.h"

namespace ge_host {

void launch_ragged_128(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st) { launch_ragged_tile<128>(p, raw, grid, st); }

}  // namespace ge_host
