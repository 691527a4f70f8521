// Guarded GEMM kernels for argument lists the fast kernels do not take (odd
// sizes, unaligned pointers, odd leading dimensions) and that are small, or
// whose fp32 rows of C are 2^24 elements and more apart under ragged tiles.
// Every global access is predicated on the M/N/K remainders and stores are
// masked (Debugging guide, checklist "Edges").  Same matrix instructions and
// the same in-register epilogue as the fast path.
#pragma once
#include "ge_device.h"

namespace ge {

// ---------------------------------------------------------------------------
// bf16, any M, N, K, lda, ldb; 2-byte aligned pointers.
// 64x64 tile, K step 32, 4 waves (2x2) of one 32x32 accumulator each.
// A is staged as [m][k], B transposed as [n][k], both padded to 40 elements so
// each lane's 8 consecutive k (16 bytes) sit in distinct banks across rows.
// ---------------------------------------------------------------------------
template <bool RAW>
__global__ void __launch_bounds__(256)
gemm_bf16_generic_kernel(const GemmParams p)
{
    constexpr int BM = 64, BN = 64, BK = 32, LD = BK + 8;
    __shared__ __attribute__((aligned(16))) uint16_t sA[BM * LD];
    __shared__ __attribute__((aligned(16))) uint16_t sB[BN * LD];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w >> 1, wn = w & 1;
    const TileCoord tc = map_block(p);
    const int m0 = tc.tm * BM, n0 = tc.tn * BN;
    const int kBegin = tc.s * p.kPerSlice;
    const int kEnd = min(p.K, kBegin + p.kPerSlice);

    const uint16_t *A = (const uint16_t *)p.A + (long long)tc.b * p.strideA;
    const uint16_t *B = (const uint16_t *)p.B + (long long)tc.b * p.strideB;

    f32x16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

    for (int k0 = kBegin; k0 < kEnd; k0 += BK) {
#pragma unroll
        for (int i = 0; i < BM * BK / 256; ++i) {
            const int e = tid + i * 256, row = e / BK, k = e % BK;
            const int m = m0 + row, kk = k0 + k;
            uint16_t v = 0;
            if (m < p.M && kk < kEnd) v = A[(long long)m * p.lda + kk];
            sA[row * LD + k] = v;
        }
#pragma unroll
        for (int i = 0; i < BK * BN / 256; ++i) {
            const int e = tid + i * 256, k = e / BN, col = e % BN;
            const int n = n0 + col, kk = k0 + k;
            uint16_t v = 0;
            if (n < p.N && kk < kEnd) v = B[(long long)kk * p.ldb + n];
            sB[col * LD + k] = v;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int kk = ks * 16 + (lane >> 5) * 8;
            bf16x8_t a = *(const bf16x8_t *)&sA[(wm * 32 + (lane & 31)) * LD + kk];
            bf16x8_t b = *(const bf16x8_t *)&sB[(wn * 32 + (lane & 31)) * LD + kk];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
        }
        __syncthreads();
    }

    float *cBase;
    long long ldc;
    if (RAW) {
        ldc = p.N;
        cBase = p.C + (long long)tc.s * p.sliceStride + (long long)tc.b * p.M * p.N;
    } else {
        ldc = p.ldc;
        cBase = p.C + (long long)tc.b * p.strideC;
    }
    const int n = n0 + wn * 32 + (lane & 31);
    if (n < p.N) {
        const float bv = (!RAW && p.bias != nullptr) ? p.bias[n] : 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (m < p.M) {
                float v = acc[r];
                if (!RAW) v = epilogue_value_rt(v, p.alpha, bv, p.act);
                cBase[(long long)m * ldc + n] = v;
            }
        }
    }
}

}  // namespace ge
