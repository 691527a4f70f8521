// Launches of gemm_bf16_ragged_kernel (gemm_ragged.h) for the storages of p.transA / p.transB: fp32 partial tiles (raw),
// else the consumer chain of p with output of p.cType.  One function per tile size and number of waves, each a
// translation unit.
#pragma once
#include <hip/hip_runtime.h>

#include "ge_device.h"

namespace ge_host {

void launch_ragged_128(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st);
void launch_ragged_128_w8(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st);
void launch_ragged_64(const ge::GemmParams &p, bool raw, dim3 grid, hipStream_t st);

}  // namespace ge_host
