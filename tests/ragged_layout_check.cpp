// Host model of how the kernel for operands of any alignment fills its LDS stages: every read lies inside the operand,
// and after the last step's shift every element of the stage that reaches a stored result is the operand's (or zero, beyond K).
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2604_01489_amd/csrc/ragged_layout.h"

using namespace ge;
static long long checked = 0;

// rowsTotal x payload elements with leading dimension ld; for STRIDED rows are k, else rows are M / N.  F32: chunks of
// four elements and 32-k steps, else of eight and 64-k steps.
template <int BX, bool STRIDED, bool F32>
void run_one(int X, int K, int ld, int kBegin, int kEnd)
{
    const int rowsTotal = STRIDED ? K : X, payload = STRIDED ? X : K;
    constexpr int E = F32 ? 4 : 8, STEP = F32 ? 32 : 64, PER_LANE = BX / 32;
    if (payload < E || kEnd <= kBegin) return;                                   // the kernels take such rows element by element, or not at all
    const long long size = (long long)(rowsTotal - 1) * ld + payload;
    auto value = [&](long long e) { return (int)(e % 65521) + 1; };
    for (int x0 = 0; x0 < X; x0 += BX) {
        const int nk = (kEnd - kBegin + STEP - 1) / STEP, left = X - x0;
        for (int t = 0; t < nk; ++t) {
            const int k0 = kBegin + t * STEP, kLeft = kEnd - k0;
            const long long base = STRIDED ? (long long)k0 * ld + x0 : (long long)x0 * ld + k0;
            std::vector<int> stage(BX * STEP, -1);
            for (int w = 0; w < 4; ++w)
                for (int lane = 0; lane < 64; ++lane)
                    for (int j = 0; j < PER_LANE; ++j) {
                        int r = 0, c = 0, slab = 0, sh = 0;
                        long long off = 0;
                        if constexpr (F32) ragged_place_f32<BX, STRIDED>(j, w, lane, r, c, slab);
                        else ragged_place<BX, STRIDED>(j, w, lane, r, c, slab);
                        if (t + 1 < nk) off = ragged_offset<STRIDED, E>(r, c, ld, left);
                        else ragged_last<STRIDED, E>(r, c, ld, left, kLeft, off, sh);
                        if (base + off < 0 || base + off + E > size) {
                            std::printf("E %d BX %d strided %d X %d K %d ld %d k [%d, %d) x0 %d step %d: read %lld of %lld\n", E, BX, STRIDED, X, K, ld, kBegin, kEnd, x0, t, base + off, size);
                            std::exit(1);
                        }
                        for (int e = 0; e < E; ++e) stage[slab * 64 * E + lane * E + e] = e + sh < E ? value(base + off + e + sh) : 0;
                    }
            for (int x = 0; x < BX && x0 + x < X; ++x)
                for (int k = 0; k < STEP; ++k) {
                    int at;
                    if (F32) at = (k / 16) * (BX * 16) + (STRIDED ? lds_b_offset<2 * BX>(k % 16, x / 4) / 4 + x % 4 : lds_a_offset(x, k % 16 / 4) / 4 + k % 4);
                    else if (STRIDED) at = (k / 32) * (BX * 32) + lds_b_offset<BX>(k % 32, x / 8) / 2 + x % 8;
                    else at = lds_a64_offset(x, k / 8) / 2 + k % 8;
                    const long long e = STRIDED ? (long long)(k0 + k) * ld + x0 + x : (long long)(x0 + x) * ld + k0 + k;
                    const int want = k0 + k < kEnd ? value(e) : 0;
                    if (stage[at] != want) {
                        std::printf("E %d BX %d strided %d X %d K %d ld %d k [%d, %d): x %d k %d holds %d, not %d\n", E, BX, STRIDED, X, K, ld, kBegin, kEnd, x0 + x, k0 + k, stage[at], want);
                        std::exit(1);
                    }
                    ++checked;
                }
        }
    }
}

template <int BX, bool STRIDED>
void run(int X, int K, int ld, int kBegin, int kEnd)
{
    run_one<BX, STRIDED, false>(X, K, ld, kBegin, kEnd);
    run_one<BX, STRIDED, true>(X, K, ld, kBegin, kEnd);
}

int main()
{
    const int sizes[] = {4, 5, 7, 8, 9, 15, 63, 64, 65, 71, 127, 128, 129, 135, 200}, pads[] = {0, 1, 3, 8};
    for (int X : sizes)
        for (int K : sizes)
            for (int pad : pads) {
                run<128, false>(X, K, K + pad, 0, K);
                run<64, false>(X, K, K + pad, 0, K);
                run<128, true>(X, K, X + pad, 0, K);
                run<64, true>(X, K, X + pad, 0, K);
                run_one<64, false, true>(X, K, K + pad, 16, K);        // fp32 slices are multiples of 16
                run_one<128, true, true>(X, K, X + pad, 16, K);
                if (K > 64) {                                  // K slices, and the ranges of a triangular operand
                    run<128, false>(X, K, K + pad, 64, K);
                    run<64, true>(X, K, X + pad, 64, K);
                    run<64, false>(X, K, K + pad, 0, 64);
                    run<128, true>(X, K, X + pad, 0, 64);
                }
            }
    // the rows of an operand stored along k may be fewer than 8, and the k rows of one stored along M or N
    for (int few : {1, 2, 7})
        for (int n : {8, 64, 131}) {
            run<128, false>(few, n, n, 0, n);
            run<64, false>(few, n, n + 1, 0, n);
            run<64, true>(n, 9, n + 1, 0, 9);
        }
    // tiles at the largest sizes: what hangs over the end does, at no sum beyond the largest int
    for (int n : {32, 64, 128, 256})
        for (long long end : {1ll, 63ll, 64ll, 255ll, 256ll, 257ll, (1ll << 31) - 257, (1ll << 31) - 256, (1ll << 31) - 129, (1ll << 31) - 64, (1ll << 31) - 1}) {
            volatile int first = (int)((end - 1) / n * n), size = (int)end;
            if (tile_inside(first, n, size) != (first + (long long)n <= end)) {
                std::printf("tile of %d at %d of %lld\n", n, first, end);
                return 1;
            }
        }
    std::printf("ragged layout ok: %lld elements\n", checked);
    return 0;
}
