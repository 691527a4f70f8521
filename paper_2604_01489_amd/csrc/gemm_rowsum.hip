// Row sum of a linear layer by its collapsed form (see include/gemm_epilogue.h):
// y = alpha * A s + t with s = the sums of B over the output dimension and t = the sum of the bias.
// Three reductions over bf16 matrices with fp32 sums in a fixed order, all bound by HBM.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/gemm_epilogue.h"
#include "ge_device.h"
#include "ge_host.h"

namespace {

using namespace ge_host;

// Rows of the matrix one block of the column-sum pass adds up: 64, or fewer where that makes too few blocks for the CUs (a
// block's rows are a chain of round trips, eight rows each: 911 x 1408, 15 blocks of 64 rows: 19.9 -> 13.7 us for both calls on 1757 rows).
constexpr int kMaxChunkRows = 64;
int col_chunk_rows(int N, int K)
{
    int rows = kMaxChunkRows;
    while (rows > 16 && (long long)ceil_div(N, rows) * ceil_div(K, 2048) < kNumCU) rows /= 2;
    return rows;
}
constexpr int kRowWaves = 16;           // waves of a block of the row pass (one staging of v per block)
constexpr int kBlockRows = 8;           // rows a block of the wide row pass takes, all in flight at once

// A streamed operand is read once and never again: the non-temporal hint keeps it from displacing
// anything in the caches, and on this part a read-only stream measured 7.1 TB/s with it against
// 6.3 TB/s without (sizes beyond the memory-side cache).
__device__ inline ge::i32x4_t load_stream16(const void *p) { return __builtin_nontemporal_load((const ge::i32x4_t *)p); }

// The same at any address (a plain load: the hint's builtin wants an aligned one).
__device__ inline ge::i32x4_t load_any16(const void *p) { return ((const ge::i32x4_any_t *)p)->v; }

__device__ inline float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

// sum over the 64 lanes of a wave, the same tree every time
__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// n terms (a power of two) added in pairs, then pairs of pairs: the halves of the range are sums of the same kind
template <int n>
__device__ inline float pair_sum(const float *t)
{
    if constexpr (n == 1) return t[0];
    else return pair_sum<n / 2>(t) + pair_sum<n / 2>(t + n / 2);
}

// sum of x[0..n) by the first 256 threads of one block: a thread adds every 256th element, then a fixed tree (x may be null: 0).  Eight loads are on their way at a time.
__device__ inline void block_vector_sum(int n, const float *__restrict__ x, float *__restrict__ out)
{
    __shared__ float part[4];
    float acc = 0.0f;
    if (x != nullptr && threadIdx.x < 256)
        for (unsigned i = threadIdx.x; i < (unsigned)n; i += 8 * 256) {
            float t[8];
#pragma unroll
            for (unsigned u = 0; u < 8; ++u) t[u] = i + 256 * u < (unsigned)n ? x[i + 256 * u] : 0.0f;
#pragma unroll
            for (unsigned u = 0; u < 8; ++u) acc = i + 256 * u < (unsigned)n ? acc + t[u] : acc;
        }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0 && threadIdx.x < 256) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (part[0] + part[1]) + (part[2] + part[3]);
}

// A vector whose sum the first block of a row pass takes on (SUM).  In a launch of its own, with one load on its way at a time, it cost the parameter call on weights K x N
// more than a launch (both calls, us, rows x inputs x outputs: 976 x 3156 x 1152 12.9 -> 11.0, 1024 x 1088 x 7805 20.5 -> 11.6; N x K, whose finish pass has the loads: 722 x 2276 x 7200 24.1 -> 19.1).
struct VectorSum {
    int n;
    const float *x;
    float *out;
};

// out[r] = scale * sum_c X[r,c] * v[c] + add[0]   (v == nullptr: ones; add == nullptr: 0)
// One wave per row at a time, a lane takes 8 consecutive columns per step (16 bytes of X) when
// VEC, single columns otherwise; v is staged in LDS once per block when it fits (`stage`), and a
// block of 16 waves walks rows with the stride of the grid so that the staging is paid once per many rows.
template <bool VEC, bool SUM>
__global__ void __launch_bounds__(kRowWaves * 64)
rows_dot_kernel(int R, int C, const uint16_t *__restrict__ X, long long ldx, const float *__restrict__ v,
                float scale, const float *__restrict__ add, float *__restrict__ out, int stage, VectorSum sum)
{
    constexpr int extra = SUM ? 1 : 0;
    const int block = (int)blockIdx.x - extra;
    if (SUM && block < 0) {
        block_vector_sum(sum.n, sum.x, sum.out);
        return;
    }
    extern __shared__ float vs[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (stage) {
        for (int c = threadIdx.x; c < C; c += kRowWaves * 64) vs[c] = v[c];
        __syncthreads();
    }
    const float *vv = stage ? vs : v;
    const float addv = add != nullptr ? add[0] : 0.0f;
    for (long long r = (long long)block * kRowWaves + w; r < R; r += (long long)((int)gridDim.x - extra) * kRowWaves) {
        const uint16_t *row = X + r * ldx;
        float acc = 0.0f;
        if (VEC) {
            const int c8 = C / 8;
#pragma unroll 4
            for (int q = lane; q < c8; q += 64) {
                const ge::i32x4_t x = *(const ge::i32x4_t *)(row + 8 * q);
                float f[8] = {bf16_lo((unsigned)x[0]), bf16_hi((unsigned)x[0]), bf16_lo((unsigned)x[1]), bf16_hi((unsigned)x[1]),
                              bf16_lo((unsigned)x[2]), bf16_hi((unsigned)x[2]), bf16_lo((unsigned)x[3]), bf16_hi((unsigned)x[3])};
                if (vv != nullptr) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc = __builtin_fmaf(f[e], vv[8 * q + e], acc);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc += f[e];
                }
            }
            // (unsigned: 64 columns on from the last of nearly 2^31 is past the largest int)
            for (unsigned c = c8 * 8 + lane; c < (unsigned)C; c += 64) {
                const float f = bf16_lo((unsigned)row[c]);
                acc = vv != nullptr ? __builtin_fmaf(f, vv[c], acc) : acc + f;
            }
        } else {
            for (unsigned c = lane; c < (unsigned)C; c += 64) {
                const float f = bf16_lo((unsigned)row[c]);
                acc = vv != nullptr ? __builtin_fmaf(f, vv[c], acc) : acc + f;
            }
        }
        acc = wave_sum(acc);
        if (lane == 0) out[r] = __builtin_fmaf(scale, acc, addv);
    }
}

// The same for matrices whose rows can be read in 16-byte pieces (not ANY: C a multiple of 8, aligned) and are at least
// 384 columns wide: a block of WAVES waves is G groups, each group takes kBlockRows
// consecutive rows; a thread owns 8 consecutive columns per sweep of 512 WAVES / G columns, holds their v in
// registers and has one 16-byte load per row in flight, all issued before the first is used.  Many
// short-lived blocks that each ask for everything up front keep more of the memory system busy than few
// long-lived waves that walk their own rows: measured on an 8192 x 8192 matrix beyond the
// memory-side cache, 23 us against 33-37 us for the kernel above.  Small blocks, because a CU that holds several is
// still reading for some while others add up, and because a small call waits for the start of its largest block: with four or eight
// waves instead of 16 both calls on 16384 x 4096 + 8192 x 4096 take 47.0 us for 56.1, on 2048 x 2048 twice 12.8 for 17.7, 8192 x
// 8192 twice 57.4 for 58.5.  Starting each block's sweeps at another column changed nothing.  Per row: a sweep's eight products, the
// sweeps, a fixed butterfly inside each wave, then the wave sums of its group added in wave order.
// ANY: rows at any address and of any length of at least 8; the chunk at a row's end is pulled back to end there and
// shifted down, which puts zeros beyond (12096 x 2205 + 2752 x 2205: 26.1 us for both calls, 50.8 by the kernel above).
template <int WAVES, int G, bool ANY, bool SUM>
__global__ void __launch_bounds__(WAVES * 64)
rows_dot_wide_kernel(int R, int C, const uint16_t *__restrict__ X, long long ldx, const float *__restrict__ v,
                     float scale, const float *__restrict__ add, float *__restrict__ out, VectorSum sum)
{
    const int block = (int)blockIdx.x - (SUM ? 1 : 0);
    if (SUM && block < 0) {
        block_vector_sum(sum.n, sum.x, sum.out);
        return;
    }
    constexpr int WG = WAVES / G;                   // waves of a group
    constexpr int SWEEP = WG * 64 * 8;              // columns a group covers in one sweep
    __shared__ float part[G * kBlockRows][WG];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int g = w / WG, wg = w % WG;
    const long long r0 = ((long long)block * G + g) * kBlockRows;
    float acc[kBlockRows];
#pragma unroll
    for (int u = 0; u < kBlockRows; ++u) acc[u] = 0.0f;
    // (unsigned: a sweep beyond the last of nearly 2^31 columns is past the largest int)
    for (unsigned first = (wg * 64 + lane) * 8; first < (unsigned)C; first += SWEEP) {
        const int c0 = (int)first;
        ge::i32x4_t x[kBlockRows];
        float vv[8];
        if constexpr (ANY) {
            // rows beyond R are the last one again: their sums are not stored
            const int at = c0 < C - 8 ? c0 : C - 8;
#pragma unroll
            for (int u = 0; u < kBlockRows; ++u) x[u] = load_any16(X + (r0 + u < R ? r0 + u : R - 1) * ldx + at);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool inside = c0 + e < C;
                vv[e] = inside ? (v != nullptr ? v[inside ? c0 + e : 0] : 1.0f) : 0.0f;
            }
            if (at != c0) {
#pragma unroll
                for (int u = 0; u < kBlockRows; ++u) x[u] = ge::shift_down_elements(x[u], c0 - at);
            }
        } else {
#pragma unroll
            for (int u = 0; u < kBlockRows; ++u) {
                x[u] = ge::i32x4_t{0, 0, 0, 0};
                if (r0 + u < R) x[u] = load_stream16(X + (r0 + u) * ldx + c0);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) vv[e] = v != nullptr ? v[c0 + e] : 1.0f;
        }
#pragma unroll
        for (int u = 0; u < kBlockRows; ++u) {
            float t = 0.0f;                             // a sweep's eight products, then the sweeps
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t = __builtin_fmaf(bf16_lo((unsigned)x[u][e]), vv[2 * e], t);
                t = __builtin_fmaf(bf16_hi((unsigned)x[u][e]), vv[2 * e + 1], t);
            }
            acc[u] += t;
        }
    }
#pragma unroll
    for (int u = 0; u < kBlockRows; ++u) {
        const float t = wave_sum(acc[u]);
        if (lane == 0) part[g * kBlockRows + u][wg] = t;
    }
    __syncthreads();
    if (threadIdx.x < G * kBlockRows) {
        const long long r = (long long)block * G * kBlockRows + threadIdx.x;      // rows of a block are consecutive
        if (r < R) {
            float t = 0.0f;
#pragma unroll
            for (int k = 0; k < WG; ++k) t += part[threadIdx.x][k];
            out[r] = __builtin_fmaf(scale, t, add != nullptr ? add[0] : 0.0f);
        }
    }
}

// partial[chunk][c] = sum over the rows of chunk `chunk` (chunkRows rows) of X[r,c]: SUBS runs of chunkRows / SUBS rows, each
// added in row order, then in pairs.  The runs are what the sizes ask for (col_chunk_rows) and SUBS is 1, unless the workspace
// holds only longer chunks: then a block adds up here, in the same pairs, the runs that cols_finish_kernel adds up
// otherwise, and the sums are the same bit for bit.
// A thread owns 8 consecutive columns (16 bytes per row; ALIGNED: rows of whole aligned pieces, by non-temporal loads; else at
// any address), or one column where rows are shorter (WIDE false).  The loads of 8 rows are issued together, ahead of the additions of the 8
// before (left to the compiler's unrolling they went out one by one behind a bounds test: 50 us for 8192 x 8192 against 23 us).  What bounds it
// is the reads in flight: two blocks of four waves on a CU.  With nothing asked for while a wave added, 5312 x 5685 + 8191 x 5685
// took 56.6 us for both calls, 47.1 now; aligned rows, 2048 x 1024 twice, 16.3 / 14.9.
template <bool WIDE, bool ALIGNED, int SUBS>
__global__ void __launch_bounds__(256)
cols_partial_kernel(int R, int C, const uint16_t *__restrict__ X, long long ldx, float *__restrict__ partial, int chunkRows)
{
    constexpr int W = WIDE ? 8 : 1, U = 8;
    const int c0 = (blockIdx.x * 256 + threadIdx.x) * W;
    if (c0 >= C) return;
    // the columns at the end of a row are read with those before them; only they are stored
    const int at = WIDE && !ALIGNED && c0 > C - 8 ? C - 8 : c0;
    const int runRows = chunkRows / SUBS, chunkEnd = min(R, (int)(blockIdx.y + 1) * chunkRows);
    float acc[SUBS][W];
#pragma unroll
    for (int q = 0; q < SUBS; ++q) {
#pragma unroll
        for (int e = 0; e < W; ++e) acc[q][e] = 0.0f;
        const int r0 = blockIdx.y * chunkRows + q * runRows, r1 = min(chunkEnd, r0 + runRows);
        if constexpr (WIDE) {
            // U rows; not whole: those beyond r1 are the last one again, and not added
            auto fetch = [&](int r, ge::i32x4_t (&x)[U], auto whole) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint16_t *src = X + (long long)(decltype(whole)::value || r + u < r1 ? r + u : r1 - 1) * ldx + at;
                    x[u] = ALIGNED ? load_stream16(src) : load_any16(src);
                }
            };
            auto add = [&](int r, const ge::i32x4_t (&x)[U], auto whole) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool inside = decltype(whole)::value || r + u < r1;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc[q][2 * e] += inside ? bf16_lo((unsigned)x[u][e]) : 0.0f;
                        acc[q][2 * e + 1] += inside ? bf16_hi((unsigned)x[u][e]) : 0.0f;
                    }
                }
            };
            constexpr std::true_type whole{};
            constexpr std::false_type part{};
            ge::i32x4_t x[2][U];
            int r = r0;
            if (r + 2 * U <= r1) {
                fetch(r, x[0], whole);
                for (; r + 4 * U <= r1; r += 2 * U) {
                    fetch(r + U, x[1], whole);
                    add(r, x[0], whole);
                    fetch(r + 2 * U, x[0], whole);
                    add(r + U, x[1], whole);
                }
                fetch(r + U, x[1], whole);
                add(r, x[0], whole);
                add(r + U, x[1], whole);
                r += 2 * U;
            }
            for (; r < r1; r += U) {
                fetch(r, x[0], part);
                add(r, x[0], part);
            }
        } else {
            for (int r = r0; r < r1; ++r) acc[q][0] += bf16_lo((unsigned)X[(long long)r * ldx + c0]);
        }
    }
#pragma unroll
    for (int e = 0; e < W; ++e) {
        float t[SUBS];
#pragma unroll
        for (int q = 0; q < SUBS; ++q) t[q] = acc[q][e];
        const int c = at + e;
        if (c >= c0 && c < C) partial[(long long)blockIdx.y * C + c] = pair_sum<SUBS>(t);
    }
}

// s[c] = sum of the chunks' partial sums; the block past the last column block adds up the bias into
// s[C].  A block covers 64 columns: 16 groups of 16 threads, a thread 4 consecutive columns (16 bytes per
// load).  Group g adds up 64-row chunks g, g + 16, ... in ascending order, eight loads in flight at a time, a chunk
// whose partial sums are of 64 / SUBS rows in pairs; then the 16 sums are added in the order of g (32 groups of 8 threads: the same 5 us, a launch and a round trip).  (One thread per column over all chunks left the pass at
// the latency of a chain of dependent loads: 10 us for 2 MB; 8 groups of single columns: 6.9 us.)
constexpr int kFinishCols = 64, kFinishWays = 16;
template <int SUBS>
__global__ void __launch_bounds__(256)
cols_finish_kernel(int C, int partials, const float *__restrict__ partial, float *__restrict__ s, int nBias,
                   const float *__restrict__ bias)
{
    if (blockIdx.x == gridDim.x - 1) {
        block_vector_sum(nBias, bias, s + C);
        return;
    }
    __shared__ float part[kFinishWays][kFinishCols];
    const int g = threadIdx.x / (kFinishCols / 4), cl = (threadIdx.x % (kFinishCols / 4)) * 4;
    const int c = blockIdx.x * kFinishCols + cl;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    // four columns by one 16-byte load at any address; those at the end of a row are read with the ones before them, and only
    // they are kept
    const bool wide = C >= 4;
    const int at = wide && c > C - 4 ? C - 4 : c;
    constexpr int U = 8 / SUBS;                           // chunks whose loads are on their way together
    for (int q0 = g; q0 * SUBS < partials; q0 += U * kFinishWays) {
        ge::i32x4_t t[U][SUBS];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int first = (q0 + u * kFinishWays) * SUBS;
#pragma unroll
            for (int i = 0; i < SUBS; ++i) t[u][i] = ge::i32x4_t{0, 0, 0, 0};
            const float *src = partial + (long long)first * C + (wide ? at : 0);
            if (wide && first + SUBS <= partials && c < C) {
#pragma unroll
                for (int i = 0; i < SUBS; ++i) t[u][i] = load_any16(src + (long long)i * C);
            } else if (c < C) {                           // the last chunk, of fewer runs
#pragma unroll
                for (int i = 0; i < SUBS; ++i)
                    if (first + i < partials) {
                        if (wide) t[u][i] = load_any16(src + (long long)i * C);
                        else
                            for (int e = 0; e < C; ++e) t[u][i][e] = (int)__float_as_uint(src[(long long)i * C + e]);
                    }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v[SUBS];
#pragma unroll
                for (int i = 0; i < SUBS; ++i) v[i] = __uint_as_float((unsigned)t[u][i][e]);
                acc[e] += pair_sum<SUBS>(v);
            }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (at + e >= c) part[g][cl + (at - c) + e] = acc[e];
    __syncthreads();
    if (threadIdx.x < kFinishCols) {
        const int cc = blockIdx.x * kFinishCols + threadIdx.x;
        if (cc < C) {
            float t = part[0][threadIdx.x];
#pragma unroll
            for (int k = 1; k < kFinishWays; ++k) t += part[k][threadIdx.x];
            s[cc] = t;
        }
    }
}

bool vec_ok(const void *base, long long ld) { return (((uintptr_t)base) & 15u) == 0 && ld % 8 == 0; }

bool rows_aligned(int C, const void *X, long long ldx) { return vec_ok(X, ldx) && C % 8 == 0; }

// The wide kernel needs enough columns to give most lanes of a wave a 16-byte piece (its narrowest sweep is 512 columns).
// Rows that are no whole aligned pieces take it only where it is the shorter call (us, one wave a row / wide):
// - at any address, from 2048 columns on (2049 x 4096 rows 25.3 / 8.8, 8191 x 8192 rows 53.4 / 30.8, 1000 x 2100 7.7 / 5.2) or 2^23 elements (911
//   columns: 8192 rows 5.5 / 6.3 or 5.7, 12288 8.1 / 7.9 or 12.5 / 7.1; 505: 16384 6.0 / 6.7, 24576 11.1 / 8.4; 1351: 8192 11.4 / 8.1).  Between, from about
//   1300 columns and 2^22.5 elements on, the line keeps some on the slower side (4096 x 1351 6.2 / 5.7, 6000 x 1351 11.0 / 6.8, 4096 x 2001 10.8 / 6.8);
// - at 16-byte addresses and of a length that is no multiple of 8, which the other kernel reads in aligned pieces but for the last
//   columns, for few long rows (5685 x 1160 8.5 / 7.0, x 4096 12.2 / 12.1; 4609 x 2048 6.5 / 6.6; 6001 x 2048 10.7 / 7.4; 30001 x 300 23.9 / 20.4; 4801 x 4096 9.6 /
//   10.6; 4301 x 2500 6.6 / 8.8).
bool rows_wide(int R, int C, const void *X, long long ldx)
{
    if (C < 384) return false;
    if (rows_aligned(C, X, ldx)) return true;
    if (vec_ok(X, ldx)) return C > 4608 && R >= 32 && R <= 2048;
    return C >= 2048 || (double)R * C >= 8.0 * 1024 * 1024;
}

// rows of X times v (or ones), on `st`; SUM: and a vector's sum
template <bool SUM>
void launch_rows_dot(int R, int C, const uint16_t *X, long long ldx, const float *v, float scale, const float *add,
                     float *out, hipStream_t st, VectorSum sum = VectorSum{0, nullptr, nullptr})
{
    constexpr unsigned extra = SUM ? 1 : 0;
    if (rows_wide(R, C, X, ldx)) {
        auto launch = [&](auto waves, auto groups) {
            constexpr int W = decltype(waves)::value, G = decltype(groups)::value;
            const dim3 blocks((unsigned)ceil_div(R, G * kBlockRows) + extra), threads(W * 64);
            if (rows_aligned(C, X, ldx)) GE_LAUNCH((rows_dot_wide_kernel<W, G, false, SUM>), blocks, threads, 0, st, R, C, X, ldx, v, scale, add, out, sum);
            else                         GE_LAUNCH((rows_dot_wide_kernel<W, G, true, SUM>), blocks, threads, 0, st, R, C, X, ldx, v, scale, add, out, sum);
        };
        using std::integral_constant;
        constexpr integral_constant<int, 4> four{};
        // Eight waves for long rows of which there are too few for two blocks to a CU (both calls, us, four / eight waves: 2048 x 4096
        // 17.1 / 16.1, 1024 x 8192 18.6 / 17.9, 2048 x 32768 39.4 / 32.8; 4096 x 8192 31.9 / 33.1, 8192 x 16384 57.6 / 71.6, 2048 x
        // 2048 13.6 / 14.5); else four, the narrowest sweep that covers a row or the whole block per row.
        // Aligned rows of a length and number that make nearly one block of 16 waves a CU, two or four rows of waves: those (the row pass, us, four or
        // eight / 16 waves: 3204 x 3072 8.1 / 8.0, 4000 x 4000 10.4 / 9.9, 3601 x 2816 8.0 / 7.9, 2077 x 3384 8.3 / 7.7, 2303 x 3752 9.0 / 8.3; 144 blocks 2300 x 2304 6.8 / 7.0;
        // 6475 x 1712 9.1 / 8.8, 8000 x 2000 10.4 / 10.0; 160 blocks 5000 x 1536 7.0 / 7.8).
        const long long of16 = C > 2048 ? ceil_div(R, 16) : ceil_div(R, 32);
        const bool one16 = rows_aligned(C, X, ldx) && C > 1024 && C <= 4096 && of16 <= kNumCU && of16 * 16 > kNumCU * (C > 2560 ? 8 : C > 2048 ? 9 : 12);
        if (one16 && C > 2048) GE_LAUNCH((rows_dot_wide_kernel<16, 2, false, SUM>), dim3((unsigned)of16 + extra), dim3(1024), 0, st, R, C, X, ldx, v, scale, add, out, sum);
        else if (one16)        GE_LAUNCH((rows_dot_wide_kernel<16, 4, false, SUM>), dim3((unsigned)of16 + extra), dim3(1024), 0, st, R, C, X, ldx, v, scale, add, out, sum);
        else if (C > 2048 && R < kBlockRows * 2 * kNumCU) launch(integral_constant<int, 8>{}, integral_constant<int, 1>{});
        else if (C <= 512)                           launch(four, integral_constant<int, 4>{});
        else if (C <= 1024)                          launch(four, integral_constant<int, 2>{});
        else                                         launch(four, integral_constant<int, 1>{});
        return;
    }
    const int stage = (v != nullptr && (size_t)C * sizeof(float) <= 48 * 1024) ? 1 : 0;
    const size_t lds = stage ? (size_t)C * sizeof(float) : 0;
    long long blocks = ((long long)R + kRowWaves - 1) / kRowWaves;
    const long long cap = 2ll * kNumCU;             // two blocks of 16 waves per CU; many rows per staging of v
    if (blocks > cap) blocks = cap;
    const dim3 threads(kRowWaves * 64);
    if (vec_ok(X, ldx)) GE_LAUNCH((rows_dot_kernel<true, SUM>), dim3((unsigned)blocks + extra), threads, lds, st, R, C, X, ldx, v, scale, add, out, stage, sum);
    else                GE_LAUNCH((rows_dot_kernel<false, SUM>), dim3((unsigned)blocks + extra), threads, lds, st, R, C, X, ldx, v, scale, add, out, stage, sum);
}

}  // namespace

extern "C" size_t gemm_rowsum_params_workspace_bytes(int N, int K, int transB)
{
    if (N < 1 || K < 1 || !transB) return 0;
    return (size_t)ceil_div(N, col_chunk_rows(N, K)) * (size_t)K * sizeof(float);
}

extern "C" ge_status_t gemm_rowsum_params_bf16(int N, int K, const uint16_t *B, int ldb, int transB,
                                               const float *bias, float *params, void *stream)
{
    return gemm_rowsum_params_bf16_ex(N, K, B, ldb, transB, bias, params, nullptr, 0, stream);
}

extern "C" ge_status_t gemm_rowsum_params_bf16_ex(int N, int K, const uint16_t *B, int ldb, int transB,
                                                  const float *bias, float *params, void *workspace,
                                                  size_t workspace_bytes, void *stream)
{
    if (!B || !params) return GE_ERR_NULL;
    if (N < 1 || K < 1) return GE_ERR_SHAPE;
    if (ldb < (transB ? K : N)) return GE_ERR_LD;
    if (transB && ceil_div(N, 64) > 65535) return GE_ERR_SHAPE;      // chunks ride on the grid's y axis
    if ((((uintptr_t)B) & 1u) || (((uintptr_t)params) & 3u) || (((uintptr_t)bias) & 3u)) return GE_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    if (!transB) {
        // B is K x N: s[k] is the sum of row k
        launch_rows_dot<true>(K, N, B, ldb, nullptr, 1.0f, nullptr, params, st, VectorSum{N, bias, params + K});
        g_last_config = "rowsum_params_rows";
    } else {
        // B is stored N x K: s[k] is the sum of column k, in two passes through the workspace.  A caller's buffer (or the
        // library's, under capture) that holds the partial sums of 64 rows a chunk is enough: where it has no room for
        // those of the shorter runs the sizes ask for, a block adds up several runs, in the order of the second pass.
        const int runRows = col_chunk_rows(N, K);
        int subs = 1, partials = ceil_div(N, runRows);
        void *ws = nullptr;
        ge_status_t rc = acquire_workspace((size_t)partials * (size_t)K * sizeof(float), workspace, workspace_bytes, st, &ws);
        while (rc == GE_ERR_WORKSPACE && runRows * subs < kMaxChunkRows) {
            subs *= 2;
            partials = ceil_div(N, runRows * subs);
            rc = acquire_workspace((size_t)partials * (size_t)K * sizeof(float), workspace, workspace_bytes, st, &ws);
        }
        if (rc != GE_OK) return rc;
        float *partial = (float *)ws;
        const dim3 grid((unsigned)ceil_div(K, 256 * (K >= 8 ? 8 : 1)), (unsigned)partials);
        auto sums = [&](auto subsC) {
            constexpr int S = decltype(subsC)::value;
            const int chunkRows = runRows * S;
            if (K < 8)                        GE_LAUNCH((cols_partial_kernel<false, false, S>), grid, dim3(256), 0, st, N, K, B, (long long)ldb, partial, chunkRows);
            else if (rows_aligned(K, B, ldb)) GE_LAUNCH((cols_partial_kernel<true, true, S>), grid, dim3(256), 0, st, N, K, B, (long long)ldb, partial, chunkRows);
            else                              GE_LAUNCH((cols_partial_kernel<true, false, S>), grid, dim3(256), 0, st, N, K, B, (long long)ldb, partial, chunkRows);
        };
        if (subs == 1)      sums(std::integral_constant<int, 1>{});
        else if (subs == 2) sums(std::integral_constant<int, 2>{});
        else                sums(std::integral_constant<int, 4>{});
        const dim3 finish((unsigned)ceil_div(K, kFinishCols) + 1);
        const int left = kMaxChunkRows / (runRows * subs);         // partial sums of a 64-row chunk
        if (left == 1)      GE_LAUNCH(cols_finish_kernel<1>, finish, dim3(256), 0, st, K, partials, (const float *)ws, params, N, bias);
        else if (left == 2) GE_LAUNCH(cols_finish_kernel<2>, finish, dim3(256), 0, st, K, partials, (const float *)ws, params, N, bias);
        else                GE_LAUNCH(cols_finish_kernel<4>, finish, dim3(256), 0, st, K, partials, (const float *)ws, params, N, bias);
        g_last_config = "rowsum_params_cols";
    }
    return ge_host::take_launch_error() == hipSuccess ? GE_OK : GE_ERR_LAUNCH;
}

extern "C" ge_status_t gemm_rowsum_bf16(int M, int K, const uint16_t *A, int lda, const float *params,
                                        float alpha, float *y, void *stream)
{
    if (!A || !params || !y) return GE_ERR_NULL;
    if (M < 1 || K < 1) return GE_ERR_SHAPE;
    if (lda < K) return GE_ERR_LD;
    if ((((uintptr_t)A) & 1u) || (((uintptr_t)params) & 3u) || (((uintptr_t)y) & 3u)) return GE_ERR_ALIGN;
    launch_rows_dot<false>(M, K, A, lda, params, alpha, params + K, y, (hipStream_t)stream);
    g_last_config = rows_wide(M, K, A, lda) ? (rows_aligned(K, A, lda) ? "rowsum_rows_wide" : "rowsum_rows_wide_any")
                                 : vec_ok(A, lda) ? "rowsum_rows_vec8" : "rowsum_rows_generic";
    return ge_host::take_launch_error() == hipSuccess ? GE_OK : GE_ERR_LAUNCH;
}
