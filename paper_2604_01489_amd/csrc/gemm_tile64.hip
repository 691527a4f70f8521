// The 64 x 128 tile (gemm_tile64_launch.h), and which calls take it or the ones for a short K.
#include "gemm_tile64_tiles.h"

namespace ge_host {

Tile64 tile64_of(const Plan &pl, const GemmParams &p, ge_plan_t plan)
{
    if ((pl.tile != TILE_128 && pl.tile != TILE_256) || pl.splitK > 1 || plan == GE_PLAN_SPLITK || p.triA != ge::TRI_NONE || opt_force_config() != FORCE_NONE || opt_eight_waves() ||
        opt_stage_k32())
        return TILE64_NO;
    return ge::tile64_kind(pl.tile == TILE_128, (long long)ceil_div(p.M, 64) * ceil_div(p.N, 128) * p.batch, p.K, p.cType == ge::DT_BF16, ceil_div(p.M, 64) % 2 != 0);
}

const char *tile64_config(Tile64 kind, int family)
{
    static const char *const names[3][3] = {{"bf16_64x128x32_w4", "bf16_64x128_k64_w4", "bf16_128x128_k64_w4"},
                                            {"conv_bf16_64x128x32_w4", "conv_bf16_64x128_k64_w4", "conv_bf16_128x128_k64_w4"},
                                            {"conv_bf16_c8_64x128x32_w4", "conv_bf16_c8_64x128_k64_w4", "conv_bf16_c8_128x128_k64_w4"}};
    return names[family][kind - TILE64_RING];
}

void launch_tile64_ring(const GemmParams &p, dim3 grid, hipStream_t st) { launch_tile64_mode<64, 1, 4, 4, 3>(p, grid, st); }

dim3 tile64_grid(GemmParams &p, bool wide)
{
    p.tilesM = ceil_div(p.M, wide ? 128 : 64);
    p.tilesN = ceil_div(p.N, 128);
    p.groupM = choose_group_m(p.tilesM, p.tilesN);
    return dim3((unsigned)((long long)p.tilesM * p.tilesN * p.batch));
}

void launch_tile64(GemmParams p, Tile64 kind, hipStream_t st)
{
    const bool wide = kind == TILE64_SHORT_WIDE;
    const dim3 grid = tile64_grid(p, wide);
    if (kind == TILE64_RING) launch_tile64_ring(p, grid, st);
    else                     launch_tile64_short(p, wide, grid, st);
}

}  // namespace ge_host
