// One group of kernel variants of the widened operator: 256 x 256 block tiles, tiles that may hang over M, N or the K range (gemm_fused_launch.h).
#include "gemm_fused_tiles.h"

namespace ge_host {

void fused_tile_256_kedge(const ge::GemmParams &p, bool k64, bool raw, dim3 grid, hipStream_t st)
{
    launch_tile_mode<256, 256, 2, 4, 2>(p, k64, raw, grid, st);
}

}  // namespace ge_host
