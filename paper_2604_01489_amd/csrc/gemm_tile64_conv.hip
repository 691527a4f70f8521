// The tiles of gemm_tile64_launch.h for the gathering convolution.
#include "gemm_bf16_fast.h"
#include "gemm_tile64_launch.h"

namespace ge_host {

namespace {

template <int BM, int WM, int WN, int NS, int PER>
void launch_conv_mode(const GemmParams &p, bool c8, dim3 grid, hipStream_t st)
{
    constexpr int threads = WM * WN * 64;
    const bool h = p.cType == ge::DT_BF16;
    if (c8) {
        if (h) GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, 2, false, ge::ACT_NONE, false, true, true, true, 2, false, NS, PER>), grid, dim3(threads), 0, st, p);
        else   GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, 2, false, ge::ACT_NONE, false, true, true, false, 2, false, NS, PER>), grid, dim3(threads), 0, st, p);
    } else {
        if (h) GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, 1, false, ge::ACT_NONE, false, true, true, true, 1, false, NS, PER>), grid, dim3(threads), 0, st, p);
        else   GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, 1, false, ge::ACT_NONE, false, true, true, false, 1, false, NS, PER>), grid, dim3(threads), 0, st, p);
    }
}

}  // namespace

void launch_tile64_conv(GemmParams p, Tile64 kind, bool c8, hipStream_t st)
{
    const bool wide = kind == TILE64_SHORT_WIDE;
    const dim3 grid = tile64_grid(p, wide);
    if (kind == TILE64_RING) launch_conv_mode<64, 1, 4, 4, 3>(p, c8, grid, st);
    else if (wide)           launch_conv_mode<128, 2, 2, 2, 3>(p, c8, grid, st);
    else                     launch_conv_mode<64, 1, 4, 2, 4>(p, c8, grid, st);
}

}  // namespace ge_host
