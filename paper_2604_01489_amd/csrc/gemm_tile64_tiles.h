// The variants of a tile of gemm_tile64_launch.h by operand storage, output type and whether K ends inside a step.
#pragma once
#include "gemm_bf16_fast.h"
#include "gemm_tile64_launch.h"

namespace ge_host {

template <int BM, int WM, int WN, int EDGE, bool H, int NS, int PER>
void launch_tile64_layout(const GemmParams &p, dim3 grid, hipStream_t st)
{
    constexpr int threads = WM * WN * 64;
    if (p.transA) {
        if (p.transB) GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, EDGE, false, ge::ACT_NONE, true, true, true, H, 0, false, NS, PER>), grid, dim3(threads), 0, st, p);
        else          GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, EDGE, false, ge::ACT_NONE, true, false, true, H, 0, false, NS, PER>), grid, dim3(threads), 0, st, p);
    } else {
        if (p.transB) GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, EDGE, false, ge::ACT_NONE, false, true, true, H, 0, false, NS, PER>), grid, dim3(threads), 0, st, p);
        else          GE_LAUNCH((ge::gemm_bf16_kernel<BM, 128, WM, WN, EDGE, false, ge::ACT_NONE, false, false, true, H, 0, false, NS, PER>), grid, dim3(threads), 0, st, p);
    }
}

template <int BM, int WM, int WN, int NS, int PER>
void launch_tile64_mode(const GemmParams &p, dim3 grid, hipStream_t st)
{
    const bool h = p.cType == ge::DT_BF16;
    if (p.K % 32 != 0) { if (h) launch_tile64_layout<BM, WM, WN, 2, true, NS, PER>(p, grid, st); else launch_tile64_layout<BM, WM, WN, 2, false, NS, PER>(p, grid, st); }
    else               { if (h) launch_tile64_layout<BM, WM, WN, 1, true, NS, PER>(p, grid, st); else launch_tile64_layout<BM, WM, WN, 1, false, NS, PER>(p, grid, st); }
}

}  // namespace ge_host
