// gemm_bf16_small_kernel: every operand storage and output mode.
#include "gemm_small.h"
#include "gemm_small_launch.h"
#include "ge_host.h"

namespace ge_host {

template <int DEPTH, bool OUTBF16>
void launch_small_mode(const GemmParams &p, int run, dim3 grid, hipStream_t st)
{
    if (p.transA) {
        if (p.transB) GE_LAUNCH((ge::gemm_bf16_small_kernel<DEPTH, true, true, OUTBF16>), grid, dim3(256), 0, st, p, run);
        else          GE_LAUNCH((ge::gemm_bf16_small_kernel<DEPTH, true, false, OUTBF16>), grid, dim3(256), 0, st, p, run);
    } else {
        if (p.transB) GE_LAUNCH((ge::gemm_bf16_small_kernel<DEPTH, false, true, OUTBF16>), grid, dim3(256), 0, st, p, run);
        else          GE_LAUNCH((ge::gemm_bf16_small_kernel<DEPTH, false, false, OUTBF16>), grid, dim3(256), 0, st, p, run);
    }
}

template <int DEPTH>
void launch_small_depth(const GemmParams &p, int run, dim3 grid, hipStream_t st)
{
    if (p.cType == ge::DT_BF16) launch_small_mode<DEPTH, true>(p, run, grid, st);
    else                        launch_small_mode<DEPTH, false>(p, run, grid, st);
}

template <int DEPTH>
void launch_small_conv_depth(const GemmParams &p, int run, dim3 grid, hipStream_t st)
{
    if (p.cType == ge::DT_BF16) GE_LAUNCH((ge::gemm_bf16_small_kernel<DEPTH, false, true, true, true>), grid, dim3(256), 0, st, p, run);
    else                        GE_LAUNCH((ge::gemm_bf16_small_kernel<DEPTH, false, true, false, true>), grid, dim3(256), 0, st, p, run);
}

void launch_small(GemmParams p, hipStream_t st)
{
    const int run = ge::small_run(p.splitK, p.kPerSlice);
    p.tilesM = ceil_div(p.M, 32);
    p.tilesN = ceil_div(p.N, 32);
    p.groupM = choose_group_m(p.tilesM, p.tilesN);
    const dim3 grid((unsigned)((long long)p.tilesM * p.tilesN * p.batch));
    if (p.convKH > 0) {
        if (p.K <= ge::SMALL_STEP) launch_small_conv_depth<1>(p, run, grid, st);
        else                       launch_small_conv_depth<2>(p, run, grid, st);
    } else if (p.K <= ge::SMALL_STEP) launch_small_depth<1>(p, run, grid, st);
    else launch_small_depth<2>(p, run, grid, st);
}

}  // namespace ge_host
