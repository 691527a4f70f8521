// Host model of a step that is not a block's last in the kernel for bf16 operands of any alignment: rows at odd elements are read
// from their second element on, moved up behind the end of the neighbouring lane's chunk, and get their first element from a
// load of its own.  Every read lies inside the operand, and what reaches a stored result is the operand's element.
// And which of the 128 x 128 tile's kernels the calls of test_gpu_ragged_rows.py take, whose names do not tell.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2604_01489_amd/csrc/ragged_layout.h"

using namespace ge;
static long long checked = 0;

// rowsTotal x payload elements with leading dimension ld, the first at element `start` of an array at a 4-byte address
template <int BX, bool STRIDED>
void run(int X, int K, int ld, int start)
{
    const int rowsTotal = STRIDED ? K : X, payload = STRIDED ? X : K;
    if (payload < 8) return;
    const long long size = (long long)(rowsTotal - 1) * ld + payload;
    auto value = [&](long long e) { return (int)(e % 65521) + 1; };
    auto fail = [&](const char *what, int x0, int t, long long at, long long of) {
        std::printf("BX %d strided %d X %d K %d ld %d start %d, x0 %d step %d: %s %lld of %lld\n", BX, STRIDED, X, K, ld, start, x0, t, what, at, of);
        std::exit(1);
    };
    for (int x0 = 0; x0 < X; x0 += BX)
        for (int t = 0; t + 1 < (K + 63) / 64; ++t) {
            const int k0 = t * 64, left = X - x0;
            const long long base = STRIDED ? (long long)k0 * ld + x0 : (long long)x0 * ld + k0;
            std::vector<int> stage(BX * 64, -1);
            for (int w = 0; w < 4; ++w) {
                for (int j = 0; j < BX / 32; ++j) {
                    int read[64][8], place[64];
                    bool odd[64];
                    for (int lane = 0; lane < 64; ++lane) {
                        const int slot = ragged_slot<BX, STRIDED>(w, lane);
                        int r = 0, c = 0, slab = 0, r0 = 0, c0 = 0, slab0 = 0;
                        ragged_place<BX, STRIDED>(j, w, slot, r, c, slab);
                        ragged_place<BX, STRIDED>(0, w, slot, r0, c0, slab0);
                        odd[lane] = (start + base + (long long)r0 * ld) & 1;      // the lane's rows alike
                        const long long o = ragged_offset<STRIDED, 8>(r, c, ld, left), at = base + o + ((start + base + o) & 1);
                        if (at < 0 || at + 8 > size) fail("read", x0, t, at, size);
                        for (int e = 0; e < 8; ++e) read[lane][e] = value(at + e);
                        place[lane] = slab * 512 + slot * 8;
                    }
                    for (int lane = 0; lane < 64; ++lane)
                        for (int e = 0; e < 8; ++e)
                            stage[place[lane] + e] = !odd[lane] ? read[lane][e] : e ? read[lane][e - 1] : lane % 16 ? read[lane - 1][7] : 0;
                    for (int i = 0; i < ragged_rows<BX, STRIDED>(); ++i) {
                        int r = 0, at = 0;
                        ragged_first<BX, STRIDED>(j, i, w, r, at);
                        const long long e = base + ragged_offset<STRIDED, 8>(r, 0, ld, left);
                        if (e < 0 || e >= size) fail("first element", x0, t, e, size);
                        if ((start | ld) & 1) stage[at / 2] = value(e);
                    }
                }
            }
            for (int x = 0; x < BX && x0 + x < X; ++x)
                for (int k = 0; k < 64; ++k) {
                    const int at = STRIDED ? (k / 32) * (BX * 32) + lds_b_offset<BX>(k % 32, x / 8) / 2 + x % 8 : lds_a64_offset(x, k / 8) / 2 + k % 8;
                    const long long e = STRIDED ? (long long)(k0 + k) * ld + x0 + x : (long long)(x0 + x) * ld + k0 + k;
                    if (stage[at] != value(e)) fail("holds another element than", x0, t, e, size);
                    ++checked;
                }
        }
}

// one pass over all of K, operands packed but for the pads, from element `start` of an aligned array; waves * 2, + 1 for one step
int variant(int M, int N, int K, int padA, int padB, int start, bool transA, bool transB)
{
    const int lda = (transA ? M : K) + padA, ldb = (transB ? K : N) + padB;
    const bool oddA = (lda | start) & 1, oddB = (ldb | start) & 1;
    const RaggedWaves v = ragged_128_waves((unsigned)((M + 127) / 128 * ((N + 127) / 128)), (K + 63) / 64 * 64, oddA, oddB, (lda & ldb) & 1, transA, transB,
                                           2.0 * (M + N) * K + 4.0 * M * N);
    return 2 * v.waves + (v.one ? 1 : 0);
}

void check_variants()
{
    enum { FOUR = 8, FOUR_ONE = 9, EIGHT = 16 };
    // of A B stored plain, B N x K, A K x M, both
    const struct { int M, N, K, padA, padB, start, want[4]; } calls[] = {
        {2049, 1543, 129, 0, 0, 1, {EIGHT, EIGHT, EIGHT, EIGHT}}, {2049, 1543, 65, 0, 0, 1, {EIGHT, EIGHT, EIGHT, EIGHT}},
        {2056, 1537, 200, 0, 0, 0, {EIGHT, EIGHT, EIGHT, EIGHT}},
        {2056, 2184, 193, 1, 3, 0, {FOUR, FOUR, EIGHT, FOUR}}, {2056, 2184, 192, 1, 4, 0, {FOUR, FOUR, FOUR, FOUR}},
        {2056, 2184, 200, 1, 3, 0, {EIGHT, EIGHT, EIGHT, EIGHT}}, {2056, 2184, 128, 0, 0, 1, {EIGHT, EIGHT, EIGHT, EIGHT}},
        {2056, 2189, 64, 0, 0, 1, {FOUR_ONE, FOUR_ONE, FOUR_ONE, FOUR_ONE}}, {2056, 2184, 33, 1, 2, 0, {FOUR_ONE, FOUR_ONE, FOUR_ONE, FOUR_ONE}},
        // every other row odd: four blocks to a CU; three steps, and two and four; 1537 k to a block, and 1536; more than 256 MB, and less
        {4097, 4097, 129, 0, 0, 0, {EIGHT, FOUR, FOUR, FOUR}}, {2049, 2047, 191, 0, 0, 0, {EIGHT, EIGHT, FOUR, EIGHT}},
        {2049, 2047, 127, 0, 0, 0, {EIGHT, EIGHT, EIGHT, EIGHT}}, {2049, 2047, 193, 0, 0, 0, {EIGHT, EIGHT, EIGHT, EIGHT}},
        {2049, 2047, 1537, 0, 0, 0, {EIGHT, FOUR, EIGHT, EIGHT}}, {2049, 2047, 1535, 0, 0, 0, {EIGHT, EIGHT, EIGHT, EIGHT}},
        {125, 42001, 3185, 0, 0, 0, {FOUR, FOUR, FOUR, FOUR}}, {125, 36001, 1535, 0, 0, 0, {EIGHT, EIGHT, EIGHT, EIGHT}}};
    for (const auto &c : calls)
        for (int s = 0; s < 4; ++s) {
            const int got = variant(c.M, c.N, c.K, c.padA, c.padB, c.start, s >= 2, s & 1);
            if (got == c.want[s]) continue;
            std::printf("%d x %d x %d, storage %d: %d waves (one step %d)\n", c.M, c.N, c.K, s, got / 2, got & 1);
            std::exit(1);
        }
}

int main()
{
    check_variants();
    for (int X : {8, 9, 15, 63, 64, 65, 71, 127, 128, 129, 135, 200, 257})
        for (int K : {65, 66, 127, 128, 129, 191, 193, 259})
            for (int pad : {0, 1, 2, 3, 8})
                for (int start : {0, 1}) {
                    run<128, false>(X, K, K + pad, start);          // (64-wide tiles have four waves, which move nothing)
                    run<128, true>(X, K, X + pad, start);
                }
    for (int few : {1, 2, 7})
        for (int start : {0, 1}) {
            run<128, false>(few, 131, 131, start);
            run<128, false>(few, 130, 131, start);
        }
    std::printf("ragged rows ok: %lld elements\n", checked);
    return 0;
}
