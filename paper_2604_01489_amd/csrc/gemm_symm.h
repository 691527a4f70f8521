// Product with a symmetric operand given by one stored triangle, for few output columns (N <= 32):
// the partial products of  S * B,  S the symmetric M x M matrix whose lower (upper) triangle is
// stored in A, with every element of the stored triangle fetched from memory once.
//
// The paper's optimisation prompt ("Rules for GEMM") names the symmetric operand as a structure to
// exploit: its reads can be reduced.  With few columns the product is a stream of A and bound by HBM,
// so halving the bytes read is what pays.  The stored triangle is cut into super-tiles of ST x ST; one
// workgroup owns one super-tile T = A[I-rows, J-columns] and uses every 128 x 128 sub-tile of it twice
// while it sits in LDS:
//     P1[rows of I] += T   * B[rows of J]        (fragments read along the rows of the image)
//     P2[rows of J] += T^T * B[rows of I]        (fragments read across them, by transposing reads)
// For a super-tile on the diagonal both products belong to the same rows, only the sub-tiles of the
// stored triangle are walked, and in the sub-tiles on the diagonal the elements of the other triangle
// (which may hold anything) are cleared in the fragments: P1 keeps the diagonal, P2 does not.
// Row block X of the result is the sum of T_s terms, T_s the number of super-tile rows: term t comes
// from super-tile (max(X, t), min(X, t)) -- its P1 if it is the super-tile's row block, its P2 if it is
// its column block.  Every term is written to the workspace W[t][batch][M][N] by exactly one
// workgroup and the terms are added in the order of t, with the consumer chain, by the second pass of
// split-K (splitk_reduce_kernel): no atomics, bitwise repeatable.  The partial results cost
// 8 N / ST bytes per byte of A (written once, read once): a quarter at N = 16 with ST = 512.
#pragma once
#include "gemm_bf16_fast.h"
#include "gemm_skinny.h"
#include "symm_layout.h"

namespace ge {

struct SymmParams {
    const void *A;             // bf16 [batch][M][lda]
    const void *B;             // bf16, K x N (ldb >= N) or, transB, N x K (ldb >= M)
    float *W;                  // [terms][batch][M][N] fp32
    int M, N, lda, ldb, transB, upper, batch;
    int tiles;                 // super-tile rows
    int past;                  // super-tiles wider than 256: their loads go past the memory-side cache
    long long bytesA;          // extent of one batch of A: ((M - 1) lda + M) * 2
};

typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;

// keep element e of a fragment register pair iff keepLo / keepHi
__device__ __forceinline__ unsigned symm_mask_pair(unsigned w, bool keepLo, bool keepHi)
{
    return w & ((keepLo ? 0x0000FFFFu : 0u) | (keepHi ? 0xFFFF0000u : 0u));
}

// Sub-tiles on their way: four, 128 KB, where a workgroup has its CU to itself; two for super-tiles of 256, which live for
// four sub-tiles, two workgroups to a CU: one's beginning and end run under the other's loads (four stages and a CU
// each: 12288 x 4 52.0 us, this 38.6).
constexpr int symm_stages(int st) { return st == 256 ? 2 : 4; }
// whether both blocks of B have a place of their own beside the stages
constexpr bool symm_own_j(int st, int np) { return symm_stages(st) * ge_symm::STAGE_BYTES + 2 * st * np * 2 <= (st == 256 ? 80 : 160) * 1024; }

// Whether a super-tile's terms leave through their image in LDS (see there), by the columns.
constexpr bool symm_image(int n) { return n > 16 && n % 4 != 0; }

// ST: side of a super-tile (a multiple of 128: 256, 512 or 768); NP: columns of the small operand's image (16 or 32);
// UPPER: the upper triangle is the stored one; BVEC: B can be read in aligned 16-byte pieces along n (N a multiple of 8, aligned,
// not transposed); IMAGE: symm_image of the call.
//
// Bound by HBM.  Room for the ring of sub-tiles: the fragments of B's rows of J, which every sub-tile row wants again, stay in
// registers.  The walk is a loop over the rows of sub-tiles (unrolled over all of them a workgroup ran through 95 KB of code
// once).  16384 x 16: 68.4 -> 59 us, launch and second pass included.
template <int ST, int NP, bool UPPER, bool BVEC, bool IMAGE>
__global__ void __launch_bounds__(256, ST == 256 ? 2 : 1)
gemm_symm_bf16_kernel(const SymmParams p)
{
    using namespace ge_symm;
    constexpr int NS = ST / SUB;            // sub-tiles per side of a super-tile
    constexpr int NJ = NP / 16;             // 16-column blocks of the result
    constexpr int KS = SUB / 32;            // 32-k steps of a sub-tile
    constexpr int SMALL_BYTES = ST * NP * 2;
    constexpr int STAGES = symm_stages(ST), LOADS = SLABS / 4;
    // stages, then B's rows of I and, where the LDS has room, its rows of J.  Else the latter pass, until their fragments are in
    // registers, through the last of four stages (BVEC) or the place of the former.
    constexpr bool OWN_J = symm_own_j(ST, NP);
    __shared__ __attribute__((aligned(1024))) char smem[STAGES * STAGE_BYTES + (OWN_J ? 2 : 1) * SMALL_BYTES];
    const unsigned ldsBase = (unsigned)(size_t)(GE_LDS char *)smem;
    const unsigned smallI = ldsBase + STAGES * STAGE_BYTES;
    const unsigned smallJ = OWN_J ? smallI + SMALL_BYTES : BVEC && STAGES == 4 ? ldsBase + (STAGES - 1) * STAGE_BYTES : smallI;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.y;

    // super-tile (a, c), a >= c, of linear index blockIdx.x = a (a + 1) / 2 + c
    unsigned a = (unsigned)((__builtin_sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
    while (a * (a + 1) / 2 > blockIdx.x) --a;
    while ((a + 1) * (a + 2) / 2 <= blockIdx.x) ++a;
    const unsigned c = blockIdx.x - a * (a + 1) / 2;
    const int I = __builtin_amdgcn_readfirstlane(UPPER ? (int)c : (int)a);     // super-tile row
    const int J = __builtin_amdgcn_readfirstlane(UPPER ? (int)a : (int)c);     // super-tile column
    const bool diag = I == J;
    // sub-tiles of the super-tile that lie inside the matrix
    const int nI = min(NS, (p.M - I * ST + SUB - 1) / SUB), nJ = min(NS, (p.M - J * ST + SUB - 1) / SUB);

    const char *gA = (const char *)p.A + (long long)b * p.M * p.lda * 2;
    const uint16_t *gB = (const uint16_t *)p.B + (long long)b * (p.transB ? (long long)p.N * p.ldb : (long long)p.M * p.ldb);

    // ---- the blocks of the small operand: its rows (k) k0 .. k0 + ST - 1, zero beyond M and beyond N --------
    // BVEC: straight into LDS, no register and no wait of its own.
    auto stage_vec = [&](unsigned dst, int k0) __attribute__((always_inline)) {
        const rsrc_words_t res = make_rsrc(gB + (long long)k0 * p.ldb, RSRC_RECORDS);
#pragma unroll
        for (int q = 0; q < SMALL_BYTES / 4096; ++q) {
            const int slab = q * 4 + w, chunk = slab * 64 + lane, kk = chunk / (NP / 8), n = chunk % (NP / 8) * 8;
            const unsigned v = k0 + kk < p.M && n < p.N ? (unsigned)kk * (unsigned)p.ldb * 2u + (unsigned)n * 2u : OOB_OFFSET;
            lds_dma16(res, dst + (unsigned)(slab * 1024), v);
        }
    };
    // Else through registers: every load of a thread is on its way before the first is used, and none sits behind a
    // test; a chunk of 8 columns is 16 bytes at whatever address, pulled back to end inside the operand, and what
    // is not of the row is masked off.  (Element by element under a test each, the two blocks of a super-tile were most of
    // the call: 9600 x 17 80.1 -> 45.2 us, 14144 x 18 126 -> 80, 5880 x 5 28.2 -> 20.6.)
    constexpr int CPR = NP / 8, PER = ST * CPR / 256;
    const long long lastChunk = (long long)(p.M - 1) * p.ldb + p.N - 8;
    auto load_small = [&](int k0, i32x4_t (&v)[PER]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int kk = (q * 256 + (int)threadIdx.x) / CPR, n = (int)threadIdx.x % CPR * 8;
            const long long want = (long long)(k0 + kk) * p.ldb + n;
            v[q] = ((const i32x4_any_t *)(gB + (want < lastChunk ? want : lastChunk)))->v;
        }
    };
    auto store_small = [&](unsigned dst, int k0, const i32x4_t (&loaded)[PER]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int kk = (q * 256 + (int)threadIdx.x) / CPR, n = (int)threadIdx.x % CPR * 8;
            const long long want = (long long)(k0 + kk) * p.ldb + n;
            const int count = k0 + kk < p.M ? p.N - n : 0;
            i32x4_t v = loaded[q];
            if (count > 0 && want > lastChunk) v = shift_down_elements(v, (int)(want - lastChunk));
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (int)symm_mask_pair((unsigned)v[e], 2 * e < count, 2 * e + 1 < count);
            *(GE_LDS i32x4_t *)(size_t)(dst + (unsigned)small_offset(NP, kk, n)) = v;
        }
    };
    // Stored N x K: 8 k of one column by a 16-byte load at whatever address (M is a multiple of 8, so none hangs over the end), all of a
    // thread's on their way before the first is used; neighbouring lanes on neighbouring columns, which is one row of the image.
    // (Element by element, 16 columns' bank conflicts a store and a round trip for every eight: 520 x 32 15.9 us, 8192 x 16 35.3, 16384 x 32
    // 130; so 12.5, 26.1 and 106.)
    auto stage_transposed = [&](unsigned dst, int k0) __attribute__((always_inline)) {
        i32x4_t v[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int id = q * 256 + (int)threadIdx.x, n = id % NP, k = k0 + id / NP * 8;
            v[q] = ((const i32x4_any_t *)(gB + (long long)min(n, p.N - 1) * p.ldb + min(k, p.M - 8)))->v;
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int id = q * 256 + (int)threadIdx.x, n = id % NP, kk = id / NP * 8;
            const bool inside = n < p.N && k0 + kk < p.M;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned w = inside ? (unsigned)v[q][e / 2] : 0u;
                *(GE_LDS unsigned short *)(size_t)(dst + (unsigned)small_offset(NP, kk + e, n)) = (unsigned short)(e & 1 ? w >> 16 : w);
            }
        }
    };

    // ---- loads of sub-tile (rs, cs) of the super-tile into ring slot st: 8 per wave ------------------------
    // (the swizzle of a slab's rows repeats every 16 rows: one lane offset, a step of 16 rows per load)
    const int row0 = slab_row(w, lane), ch0 = slab_chunk(w, lane);
    const unsigned voff0 = (unsigned)row0 * (unsigned)p.lda * 2u + (unsigned)ch0 * 16u, rows16 = 32u * (unsigned)p.lda;
    auto issue_sub = [&](int rs, int cs, int st) __attribute__((always_inline)) {
        const int r0 = I * ST + rs * SUB, c0 = J * ST + cs * SUB;
        const long long origin = ((long long)r0 * p.lda + c0) * 2;
        // rows beyond the matrix are beyond the resource's end
        const rsrc_words_t res = make_rsrc(gA + origin, records_left(p.bytesA, origin));
        const unsigned v = c0 + ch0 * 8 >= p.M ? OOB_OFFSET : voff0, dst = ldsBase + (unsigned)(st * STAGE_BYTES + w * 1024);
#pragma unroll
        for (int q = 0; q < LOADS; ++q) {
            if (ST > 256 && p.past) lds_dma16_nt(res, dst + (unsigned)(q * 4096), v + (unsigned)q * rows16);
            else                   lds_dma16(res, dst + (unsigned)(q * 4096), v + (unsigned)q * rows16);
        }
    };

    // fragment of a small-operand image: the 32 k from kBase, column block j
    auto small_frag = [&](unsigned img, int kBase, int j) __attribute__((always_inline)) {
        const GE_LDS char *p0 = (const GE_LDS char *)(size_t)(img + (unsigned)small_frag_offset(NP, kBase, j, lane, 0));
        const GE_LDS char *p1 = (const GE_LDS char *)(size_t)(img + (unsigned)small_frag_offset(NP, kBase, j, lane, 1));
        short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)p0);
        short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)p1);
        return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    auto lds_barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // A sub-tile on the diagonal: the other triangle, which may hold anything, is cleared in the image, before the multiply of P1;
    // and the diagonal itself, which belongs to P1, before that of P2.
    auto clear_triangle = [&](unsigned img) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < SUB * SUB / 8 / 256; ++q) {
            const int id = q * 256 + (int)threadIdx.x, r = id >> 4, c = id & 15;
            if (UPPER ? c < r >> 3 : c > r >> 3) *(GE_LDS i32x4_t *)(size_t)(img + (unsigned)image_offset(r, c)) = i32x4_t{0, 0, 0, 0};
        }
        const int r = (int)threadIdx.x;                  // the chunk of its row that the diagonal crosses
        if (r < SUB) {
            GE_LDS i32x4_t *const at = (GE_LDS i32x4_t *)(size_t)(img + (unsigned)image_offset(r, r >> 3));
            i32x4_t v = *at;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c0 = (r & ~7) + 2 * e, c1 = c0 + 1;
                v[e] = (int)symm_mask_pair((unsigned)v[e], UPPER ? c0 >= r : c0 <= r, UPPER ? c1 >= r : c1 <= r);
            }
            *at = v;
        }
        lds_barrier();
    };
    auto clear_diagonal = [&](unsigned img) __attribute__((always_inline)) {
        lds_barrier();
        const int r = (int)threadIdx.x;
        if (r < SUB) *(GE_LDS short *)(size_t)(img + (unsigned)(image_offset(r, r >> 3) + (r & 7) * 2)) = 0;
        lds_barrier();
    };

    // ---- the walk: the sub-tiles row by row, a ring of them on their way ------------------------------------
    // On the diagonal of the matrix only the stored triangle's: columns 0 .. u of sub-tile row u, or (upper) u .. nJ - 1.
    auto first_of = [&](int u) { return UPPER && diag ? u : 0; };
    auto last_of = [&](int u) { return !UPPER && diag ? u : nJ - 1; };
    // Past its end nothing is loaded: a super-tile of 256 is four sub-tiles, and the two empty ones behind them cost as much of the vector
    // cache's time as these did.  With them, a barrier behind every sub-tile and all of a diagonal sub-tile read and written again for its
    // other triangle 512 x 16 took 10.3 us, 1464 x 4 10.7, 3472 x 1 12.2; now 9.3, 9.5 and 11.0.
    int pu = 0, pv = 0;                                  // the next sub-tile to load
    int ahead = 0;                                       // sub-tiles on their way
    auto issue_next = [&](int st) __attribute__((always_inline)) {
        if (pu >= nI) return;
        issue_sub(pu, pv, st);
        ++ahead;
        if (pv == last_of(pu)) { ++pu; pv = first_of(pu); }
        else ++pv;
    };
    // the first sub-tile on its way has landed (the loads complete in order), every wave's part of it
    auto wait_first = [&] __attribute__((always_inline)) {
        if (ahead >= STAGES)               asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 1) * LOADS) : "memory");
        else if (STAGES > 2 && ahead == 3) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * LOADS) : "memory");
        else if (STAGES > 2 && ahead == 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LOADS) : "memory");
        else                               asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        --ahead;
    };
    static_assert(STAGES == 2 || STAGES == 4, "a wait for each number of sub-tiles on their way");
    bf16x8_t fbJ[NS * KS][NJ];
    auto read_fragments_of_J = [&] __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NS * KS; ++k)
#pragma unroll
            for (int j = 0; j < NJ; ++j) fbJ[k][j] = small_frag(smallJ, 32 * k, j);
    };
    if constexpr (BVEC && !OWN_J && STAGES == 2) {
        // (through registers at any address, as it was without this: 520 x 24 11.5 us, 6656 x 24 21.3, 12288 x 32 62.8; so 10.4, 19.7 and 60.5)
        stage_vec(smallJ, J * ST);
        issue_next(0);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LOADS) : "memory");
        read_fragments_of_J();
        lds_barrier();
        stage_vec(smallI, I * ST);
        issue_next(1);
        if (ahead == 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LOADS) : "memory");
        else            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    } else if constexpr (BVEC) {
        constexpr int FIRST = OWN_J ? STAGES : STAGES - 1;
        stage_vec(smallJ, J * ST);
        stage_vec(smallI, I * ST);
#pragma unroll
        for (int t = 0; t < FIRST; ++t) issue_next(t);
        // both blocks of B have landed
        if (ahead == FIRST) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(FIRST * LOADS) : "memory");
        else                asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        read_fragments_of_J();
        if constexpr (!OWN_J) {
            lds_barrier();
            issue_next(STAGES - 1);
        }
    } else if (!p.transB) {
        i32x4_t vJ[PER], vI[PER];
        // (the wait for the registers is one for whatever else is on its way by then: half of the stages' loads follow it)
#pragma unroll
        for (int t = 0; t < STAGES / 2; ++t) issue_next(t);
        load_small(J * ST, vJ);
        load_small(I * ST, vI);
        store_small(smallJ, J * ST, vJ);
        if constexpr (!OWN_J) {
            lds_barrier();
            read_fragments_of_J();
            lds_barrier();
        }
        store_small(smallI, I * ST, vI);
#pragma unroll
        for (int t = STAGES / 2; t < STAGES; ++t) issue_next(t);
        lds_barrier();
        if constexpr (OWN_J) read_fragments_of_J();
    } else {
#pragma unroll
        for (int t = 0; t < STAGES / 2; ++t) issue_next(t);
        stage_transposed(smallJ, J * ST);
        if constexpr (!OWN_J) {
            lds_barrier();
            read_fragments_of_J();
            lds_barrier();
        }
        stage_transposed(smallI, I * ST);
#pragma unroll
        for (int t = STAGES / 2; t < STAGES; ++t) issue_next(t);
        lds_barrier();
        if constexpr (OWN_J) read_fragments_of_J();
    }

    f32x4_t acc1[NS][2][NJ], acc2[NS][2][NJ];    // P1 of sub-tile row s, P2 of sub-tile column s
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) { acc1[s][i][j][r] = 0.0f; acc2[s][i][j][r] = 0.0f; }

    int slot = 0;
#pragma unroll 1
    for (int u = 0; u < nI; ++u) {
        bf16x8_t fbI[KS][NJ];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < NJ; ++j) fbI[ks][j] = small_frag(smallI, u * SUB + 32 * ks, j);
        f32x4_t run[2][NJ];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) run[i][j][r] = 0.0f;
        const int first = first_of(u), last = last_of(u);
#pragma unroll
        for (int v = 0; v < NS; ++v) {
            if (v < first || v > last) continue;
            wait_first();
            const unsigned img = ldsBase + (unsigned)(slot * STAGE_BYTES);
            const bool onDiag = diag && u == v;
            if (onDiag) clear_triangle(img);
            // ---- P1: rows 32 w + 16 i + l%16 of the sub-tile, k = its columns 32 ks + 8 (l/16) + e
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const bf16x8_t fa = *(const GE_LDS bf16x8_t *)(size_t)(img + (unsigned)row_frag_offset(32 * w + 16 * i, ks, lane));
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        run[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fbJ[v * KS + ks][j], fa, run[i][j], 0, 0, 0);
                }
            if (onDiag) clear_diagonal(img);
            // ---- P2: output rows = columns 32 w + 16 i + l%16 of the sub-tile, k = its rows 32 ks + 8 (l/16) + e
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const GE_LDS char *p0 = (const GE_LDS char *)(size_t)(img + (unsigned)col_frag_offset(32 * w + 16 * i, ks, lane, 0));
                    const GE_LDS char *p1 = (const GE_LDS char *)(size_t)(img + (unsigned)col_frag_offset(32 * w + 16 * i, ks, lane, 1));
                    const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)p0);
                    const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((GE_LDS short4_t *)p1);
                    const bf16x8_t fa = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc2[v][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fbI[ks][j], fa, acc2[v][i][j], 0, 0, 0);
                }
            if (pu < nI) {
                lds_barrier();                           // every wave is done with the slot
                issue_next(slot);
            }
            slot = slot == STAGES - 1 ? 0 : slot + 1;
        }
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc1[s][i][j][r] = s == u ? run[i][j][r] : acc1[s][i][j][r];
    }
    if (diag) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc1[s][i][j][r] += acc2[s][i][j][r];
    }

    // ---- the terms: P1 is term J of row block I, P2 term I of row block J; on the diagonal their sum is term I of row
    // block I.  The rows of a term's block are one run of memory.  Register r of lane l is row l%16, column 4 (l/16) + r of a
    // 16 x 16 block (the small operand's fragments are the first operand of the matrix instruction): up to 16 columns, or a multiple of 4, leave
    // straight from the registers, 16 bytes a lane at whatever 4-byte address and what is behind the last whole four by one store more; with others, and
    // most of the lanes' pieces across two lines, the run leaves through an image of it in LDS, 1 KB a wave instruction (straight / image: 8192 x
    // 27 34.4 / 32.6 us, 12288 x 31 60.9 / 58.5, 8192 x 17 31.1 / 30.8, 520 x 21 11.7 / 12.4; 9736 x 9 29.4 / 30.8, 14336 x 13 54.0 / 56.6, 8192 x 9 25.3 / 25.9,
    // 520 x 9 9.4 / 10.0, 16384 x 9 62.6 / 62.1; before, in 4-byte stores, 9736 x 9 30.2, x 5 28.2, now 27.8).  A kernel of its own for either way: with the image's code
    // in it the straight stores took longer, too (9736 x 1 26.9 / 27.7).  (P1 row by row inside the walk, for half the
    // stores to be over by its end: 16384 x 16 58.3 -> 61.8 us, the waits for the loads then wait for the stores.)
    const unsigned pitch = (unsigned)p.N * 4u;
    const int col = 4 * (lane >> 4);
    auto term_rows = [&](int rowBlock, int term) { return (char *)(p.W + ((long long)term * p.batch + b) * p.M * p.N + (long long)rowBlock * ST * p.N); };
    auto bytes_of = [&](int rowBlock) { return min(ST, p.M - rowBlock * ST) * p.N * 4; };      // a multiple of 32: M is one of 8
    if constexpr (!IMAGE) {
        auto store = [&](const f32x4_t (&acc)[NS][2][NJ], int rowBlock, int term) __attribute__((always_inline)) {
            // rows beyond the matrix are beyond the resource's end, quads not whole out of any range; the columns behind the last whole one by
            // a store of their own
            const buffer_t rows = __builtin_amdgcn_make_buffer_rsrc(term_rows(rowBlock, term), 0, bytes_of(rowBlock), 0x00020000);
            const unsigned at = (unsigned)(32 * w + (lane & 15)) * pitch + 4u * (unsigned)col;
            auto offset = [&](int s, int i, int c) { return (int)(col + c + 3 < p.N ? at + (unsigned)(s * SUB + 16 * i) * pitch + 4u * c : OOB_OFFSET); };
            if (p.N > 3) {
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[s][i][j]), rows, offset(s, i, 16 * j), 0, 0);
            }
            if (const int left = p.N & 3; NP == 16 && left) {
                const bool mine = col == (p.N & 12);
                auto tail = [&](int s, int i) { return (int)(mine ? at + (unsigned)(s * SUB + 16 * i) * pitch : OOB_OFFSET); };
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const u32x4_t v = __builtin_bit_cast(u32x4_t, acc[s][i][0]);
                        if (left == 1)      __builtin_amdgcn_raw_buffer_store_b32(v[0], rows, tail(s, i), 0, 0);
                        else if (left == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_shufflevector(v, v, 0, 1), rows, tail(s, i), 0, 0);
                        else                __builtin_amdgcn_raw_buffer_store_b96(__builtin_shufflevector(v, v, 0, 1, 2), rows, tail(s, i), 0, 0);
                    }
            }
        };
        store(acc1, I, J);
        if (!diag) store(acc2, J, I);
        return;
    }
    lds_barrier();                                       // every wave is done with the stages
    constexpr int IMAGE_BYTES = ST * NP * 4;
    static_assert(2 * IMAGE_BYTES <= STAGES * STAGE_BYTES + SMALL_BYTES, "both terms' images fit");
    auto put = [&](unsigned image, const f32x4_t (&acc)[NS][2][NJ]) __attribute__((always_inline)) {
        const unsigned at = image + (unsigned)(32 * w + (lane & 15)) * pitch + 4u * (unsigned)col;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (16 * j + col + r < p.N) {
#pragma unroll
                    for (int s = 0; s < NS; ++s)
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            *(GE_LDS float *)(size_t)(at + (unsigned)(s * SUB + 16 * i) * pitch + 64u * j + 4u * r) = acc[s][i][j][r];
                }
    };
    put(ldsBase, acc1);
    if (!diag) put(ldsBase + IMAGE_BYTES, acc2);
    lds_barrier();
    auto send = [&](unsigned image, int rowBlock, int term) {
        char *dst = term_rows(rowBlock, term);
        const int bytes = bytes_of(rowBlock);
#pragma unroll 4
        for (int at = (int)threadIdx.x * 16; at < bytes; at += 4096) *(i32x4_t *)(dst + at) = *(const GE_LDS i32x4_t *)(size_t)(image + (unsigned)at);
    };
    send(ldsBase, I, J);
    if (!diag) send(ldsBase + IMAGE_BYTES, J, I);
}

}  // namespace ge
