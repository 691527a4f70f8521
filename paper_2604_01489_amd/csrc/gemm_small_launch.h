// Launch of gemm_bf16_small_kernel (gemm_small.h) for the storages of p.transA / p.transB and the output type of p.cType: p.tilesM, p.tilesN and p.groupM
// are set here, p.splitK and p.kPerSlice are the plan's (they say how long a chain of sums may be).
#pragma once
#include <hip/hip_runtime.h>

#include "ge_device.h"

namespace ge_host {

void launch_small(ge::GemmParams p, hipStream_t st);

}  // namespace ge_host
