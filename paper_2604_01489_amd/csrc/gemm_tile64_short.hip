// K <= 64 in one load phase, on 64 x 128 and 128 x 128 tiles (gemm_tile64_launch.h).
#include "gemm_tile64_tiles.h"

namespace ge_host {

void launch_tile64_short(const GemmParams &p, bool wide, dim3 grid, hipStream_t st)
{
    if (wide) launch_tile64_mode<128, 2, 2, 2, 3>(p, grid, st);
    else      launch_tile64_mode<64, 1, 4, 2, 4>(p, grid, st);
}

}  // namespace ge_host
