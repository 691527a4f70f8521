// Split-K second pass: the slices' partial sums W[slice][batch][M][N] added in ascending order by one thread per VEC
// consecutive outputs (no atomics: bitwise repeatable; optimisation prompt, GEMM list item 7), then the epilogue: PLAIN
// scale, bias and activation, else the run-time consumer chain.
//
// Bound by the partial tiles' way from the caches: VEC = 4 (N a multiple of 4) reads them 16 bytes a lane, eight slices on
// their way at a time, and the position of an output is a shift and a compare (one output a lane, found by two 64-bit
// divisions, took 17.0 us for 16 slices of a 1024 x 1024 result with an fp32 residual, 4.2 TB/s; this 13.3, 5.4 TB/s).
#pragma once
#include "gemm_fused.h"

namespace ge {

// lgLanes: 2^lgLanes lanes share a row, 256 >> lgLanes rows a block (the host picks the smallest power of two that spans
// N, at most a wave); blockIdx.x along a row, blockIdx.y over rows
template <bool PLAIN, int VEC>
__global__ void __launch_bounds__(256)
splitk_reduce_kernel(const GemmParams p, const float *__restrict__ W, int lgLanes)
{
    static_assert(VEC == 1 || VEC == 4, "one output, or four with 16-byte loads");
    typedef __attribute__((ext_vector_type(VEC))) float vec_t;
    const int n = (int)((blockIdx.x << lgLanes) + (threadIdx.x & ((1u << lgLanes) - 1u))) * VEC;
    if (n >= p.N) return;
    const long long rows = (long long)p.batch * p.M;
    const int perBlock = 256 >> lgLanes;
    float bias[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) bias[v] = p.bias != nullptr ? p.bias[n + v] : 0.0f;
    for (long long row = (long long)blockIdx.y * perBlock + (threadIdx.x >> lgLanes); row < rows; row += (long long)gridDim.y * perBlock) {
        const long long b = p.batch == 1 ? 0 : row / p.M;
        const int m = (int)(row - b * p.M);
        const float *src = W + row * p.N + n;
        float sum[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) sum[v] = 0.0f;
        for (int i0 = 0; i0 < p.splitK; i0 += 8) {
            // slices beyond the last are the last one again, and not added: no load behind a branch
            vec_t t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = *(const vec_t *)(src + (long long)(i0 + u < p.splitK ? i0 + u : p.splitK - 1) * p.sliceStride);
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int v = 0; v < VEC; ++v) sum[v] += i0 + u < p.splitK ? t[u][v] : 0.0f;
        }
        const long long at = b * p.strideC + (long long)m * p.ldc + n;
        if constexpr (PLAIN) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) sum[v] = epilogue_value_rt(sum[v], p.alpha, bias[v], p.act);
        } else {
            const float rs = p.rowScale != nullptr ? p.rowScale[m] : 1.0f;
            float res[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) res[v] = 0.0f;
            if (p.R != nullptr) {
                const long long rAt = b * p.strideR + (long long)m * p.ldr + n;
                if constexpr (VEC == 4) {
                    if (p.rType == DT_BF16) {
                        const u32x2_t t = ((const u32x2_any_t *)((const unsigned short *)p.R + rAt))->v;
                        res[0] = bf16_bits_as_f32(t[0] & 0xFFFFu);
                        res[1] = bf16_bits_as_f32(t[0] >> 16);
                        res[2] = bf16_bits_as_f32(t[1] & 0xFFFFu);
                        res[3] = bf16_bits_as_f32(t[1] >> 16);
                    } else {
                        const i32x4_t t = ((const i32x4_any_t *)((const float *)p.R + rAt))->v;
#pragma unroll
                        for (int v = 0; v < 4; ++v) res[v] = __uint_as_float((unsigned)t[v]);
                    }
                } else {
                    res[0] = load_as_f32(p.R, rAt, p.rType);
                }
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) sum[v] = fused_value(p, sum[v], rs, bias[v], res[v]);
        }
        if constexpr (VEC == 4) {
            if (!PLAIN && p.cType == DT_BF16) {
                u32x2_t t;
                t[0] = pack_bf16_pair(sum[0], sum[1]);
                t[1] = pack_bf16_pair(sum[2], sum[3]);
                ((u32x2_any_t *)((unsigned short *)p.C + at))->v = t;
            } else {
                i32x4_t t;
#pragma unroll
                for (int v = 0; v < 4; ++v) t[v] = (int)__float_as_uint(sum[v]);
                ((i32x4_any_t *)((float *)p.C + at))->v = t;
            }
        } else if constexpr (PLAIN) {
            p.C[at] = sum[0];
        } else {
            store_as(p.C, at, p.cType, sum[0]);
        }
    }
}

}  // namespace ge
