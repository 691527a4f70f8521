// The variants of gemm_bf16_ragged_kernel by operand storage and output mode, for one tile size and number of waves; ONE: K slices of one step at most.
#pragma once
#include "gemm_ragged.h"
#include "gemm_ragged_launch.h"
#include "ge_host.h"

namespace ge_host {

template <int BT, int NW, int MODE, bool ONE>
void launch_ragged_mode(const GemmParams &p, dim3 grid, hipStream_t st)
{
    if (p.transA) {
        if (p.transB) GE_LAUNCH((ge::gemm_bf16_ragged_kernel<BT, NW, true, true, MODE, ONE>), grid, dim3(NW * 64), 0, st, p);
        else          GE_LAUNCH((ge::gemm_bf16_ragged_kernel<BT, NW, true, false, MODE, ONE>), grid, dim3(NW * 64), 0, st, p);
    } else {
        if (p.transB) GE_LAUNCH((ge::gemm_bf16_ragged_kernel<BT, NW, false, true, MODE, ONE>), grid, dim3(NW * 64), 0, st, p);
        else          GE_LAUNCH((ge::gemm_bf16_ragged_kernel<BT, NW, false, false, MODE, ONE>), grid, dim3(NW * 64), 0, st, p);
    }
}

template <int BT, int NW, bool ONE>
void launch_ragged_tile(const GemmParams &p, bool raw, dim3 grid, hipStream_t st)
{
    if (raw) launch_ragged_mode<BT, NW, 0, ONE>(p, grid, st);
    else if (p.cType == ge::DT_BF16) launch_ragged_mode<BT, NW, 2, ONE>(p, grid, st);
    else launch_ragged_mode<BT, NW, 1, ONE>(p, grid, st);
}

}  // namespace ge_host
