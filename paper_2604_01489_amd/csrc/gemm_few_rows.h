// A few rows through a linear layer: C[M, N] = A[M, K] B with M <= 32 and B stored N x K (weights as they are kept), and the
// whole consumer chain.  One read of the weights, bound by HBM: the tall-skinny kernel (gemm_skinny.h) with the weights as
// its tall operand and the rows of A, which run along k like theirs, as its skinny one.
//
// A workgroup owns 32 rows of the weights (32 columns of C) and every row of A, and walks K in stages of 128 through a ring
// of eight (seven on their way; four where the workgroups are more than the CUs, so that two or three share one), both
// operands by direct-to-LDS loads in 256-byte row pieces, the weights with the non-temporal hint; each workgroup starts its walk at another stage.  Four waves: two blocks of 16 weight rows x two halves
// of a stage's k; the halves are added through LDS in a fixed order, then the chain, 32 consecutive columns of a row of C
// at a time.  A wave adds in runs of four stages (256 of its k, eight matrix instructions) and the runs' sums in turn: one
// chain over all of its k was less exact than the tiles' K slices, which are chains of 512 k or more (error
// against 64 bits, slices / one chain / runs: 1.30e-7 / 1.86e-7 / 9.8e-8 at 16 x 8192 x 2048, 2.73e-7 / 3.97e-7 / 1.18e-7 at
// 16 x 8192 x 8192, 3.52e-7 / 5.73e-7 / 1.40e-7 at 5 x 6144 x 16384).  The runs take no time at 16 x 8192 x 8192 (22.7 -> 22.5
// us) and 8.7 -> 9.2 us at 12 x 2808 x 2880, 88 workgroups; their end must not be a branch inside the loop over the stages, which
// copies the accumulators in every stage (23.5 and 10.1 us).
// (Weights straight from memory into the fragments' registers, 16 rows of 64 bytes per load instruction and no LDS, were slower:
// 35.9 us at 16 x 8192 x 8192, the 128 x 128 tile with K slices 38.4, this 22.5: 6.0 TB/s, launch included.  32 rows 38.4 -> 25.2.
// An image of 64 rows, six stages deep, was built and taken out:
// 64 x 8192 x 8192 39.8 -> 33.3 us, but 63 x 10432 x 6024, 326 workgroups, 47.2 -> 58.4.)
#pragma once
#include "gemm_fused.h"
#include "gemm_skinny.h"

namespace ge {

// MP: rows of the image of A (16 or 32); STAGES: depth of the ring.
template <int MP, int STAGES>
__global__ void __launch_bounds__(256)
gemm_few_rows_kernel(const GemmParams p)
{
    using namespace ge_skinny;
    constexpr int NJ = MP / 16, S_BYTES = MP * A_ROW_BYTES, S_SLABS = S_BYTES / 1024, STAGE = A_BYTES + S_BYTES;
    constexpr int LOADS = A_SLABS / 4 + S_SLABS / 4;       // loads per wave and stage
    constexpr int RUN = 4;                                 // stages whose products are one chain of additions
    static_assert((STAGES - 2) * LOADS <= 63 && S_SLABS % 4 == 0, "range of the load counter; the loads divide over the waves");
    __shared__ __attribute__((aligned(1024))) char smem[STAGES * STAGE];
    const unsigned ldsBase = (unsigned)(size_t)(GE_LDS char *)smem;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = w & 1, kh = w >> 1;                   // block of 16 weight rows, half of the stage's k
    const int n0 = (int)blockIdx.x * BM, b = (int)blockIdx.y;
    // a lower triangular A is zero from column M on: the stages beyond add nothing
    const int steps = ((p.triA == TRI_LOWER ? min(p.K, p.M) : p.K) + KS - 1) / KS;

    const long long offW = 2 * ((long long)b * p.strideB + (long long)n0 * p.ldb);
    const long long offS = 2 * ((long long)b * p.strideA);
    const char *gW = (const char *)p.B + offW, *gS = (const char *)p.A + offS;

    // per-lane offsets within a stage's piece of the weights and of A, and the lane's first k in it
    unsigned voffW[A_SLABS / 4], voffS[S_SLABS / 4];
    int kW[A_SLABS / 4], kS[S_SLABS / 4];
#pragma unroll
    for (int q = 0; q < A_SLABS / 4; ++q) {
        const int row = a_slab_row(q * 4 + w, lane), ch = a_slab_chunk(q * 4 + w, lane);
        voffW[q] = n0 + row < p.N ? (unsigned)row * (unsigned)p.ldb * 2u + (unsigned)ch * 16u : OOB_OFFSET;
        kW[q] = ch * 8;
    }
#pragma unroll
    for (int q = 0; q < S_SLABS / 4; ++q) {
        const int row = a_slab_row(q * 4 + w, lane), ch = a_slab_chunk(q * 4 + w, lane);
        voffS[q] = row < p.M ? (unsigned)row * (unsigned)p.lda * 2u + (unsigned)ch * 16u : OOB_OFFSET;
        kS[q] = ch * 8;
    }
    const int rot = steps > 1 ? (int)((blockIdx.x * 5u + blockIdx.y) % (unsigned)steps) : 0;
    // the t0-th stage of this workgroup's walk into a ring slot; past the end of the walk through an empty resource
    auto issue = [&](int t0, int slot) __attribute__((always_inline)) {
        const bool live = t0 < steps;
        const int t = live ? (t0 + rot >= steps ? t0 + rot - steps : t0 + rot) : 0;
        const long long step = (long long)t * (KS * 2);
        const rsrc_words_t rW = make_rsrc(gW + step, live ? records_left(p.bytesB, offW + step) : 0u);
        const rsrc_words_t rS = make_rsrc(gS + step, live ? records_left(p.bytesA, offS + step) : 0u);
        const int kLeft = p.K - t * KS;        // valid k in this stage
        const unsigned dst = ldsBase + (unsigned)(slot * STAGE);
#pragma unroll
        for (int q = 0; q < A_SLABS / 4; ++q)
            lds_dma16_nt(rW, dst + (unsigned)((q * 4 + w) * 1024), kW[q] >= kLeft ? OOB_OFFSET : voffW[q]);
#pragma unroll
        for (int q = 0; q < S_SLABS / 4; ++q)
            lds_dma16(rS, dst + (unsigned)(A_BYTES + (q * 4 + w) * 1024), kS[q] >= kLeft ? OOB_OFFSET : voffS[q]);
    };

    f32x4_t acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[j][r] = 0.0f;

#pragma unroll
    for (int t = 0; t < STAGES - 1; ++t) issue(t, t);
    int slot = 0;                                        // of stage t: t % STAGES
    for (int t0 = 0; t0 < steps; t0 += RUN) {
        f32x4_t run[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) run[j][r] = 0.0f;
        const int end = min(steps, t0 + RUN);
        for (int t = t0; t < end; ++t) {
            // stage t has landed, and every wave is past the multiply of t - 1, whose ring slot is refilled now
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((STAGES - 2) * LOADS) : "memory");
            issue(t + STAGES - 1, slot == 0 ? STAGES - 1 : slot - 1);
            const unsigned img = ldsBase + (unsigned)(slot * STAGE);
            slot = slot == STAGES - 1 ? 0 : slot + 1;
#pragma unroll
            for (int ks = 0; ks < KS / 64; ++ks) {       // this wave's half of the stage, 32 k at a time
                const int kk = kh * (KS / 2) + 32 * ks;
                const bf16x8_t fw = *(const GE_LDS bf16x8_t *)(size_t)(img + (unsigned)ge_skinny::a_frag_offset(16 * rg, kk, lane));
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const bf16x8_t fs = *(const GE_LDS bf16x8_t *)(size_t)(img + (unsigned)(A_BYTES + ge_skinny::a_frag_offset(16 * j, kk, lane)));
                    run[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw, fs, run[j], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[j][r] += run[j][r];
    }
    // the empty loads of the stages past the end have retired; every wave is done with the ring
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // sums[half][m][n]: register r of lane l is weight row 16 rg + 4 (l/16) + r and row 16 j + l%16 of A
    GE_LDS float *sums = (GE_LDS float *)(GE_LDS char *)smem;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        *(GE_LDS f32x4_t *)(sums + ((kh * MP + 16 * j + (lane & 15)) * BM + 16 * rg + 4 * (lane >> 4))) = acc[j];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MP * BM / 256; ++q) {
        const int o = q * 256 + (int)threadIdx.x, m = o / BM, n = n0 + o % BM;
        const float v = sums[o] + sums[MP * BM + o];     // first half + second half, always in this order
        if (m < p.M && n < p.N) fused_store(p, b, m, n, v);
    }
}

}  // namespace ge
