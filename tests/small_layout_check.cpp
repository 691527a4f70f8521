// Host model of how the kernel of few output tiles fills its LDS stages and reads its fragments: every read lies inside the operand, every
// element of a step is where the fragment of its row and k is read, and which products take the kernel (the sizes of test_gpu_small.py among them).
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2604_01489_amd/csrc/small_layout.h"

using namespace ge;
static long long checked = 0;

template <bool STRIDED>
void run(int X, int K, int ld)
{
    constexpr int BX = 32, NW = 4, E = 8;
    const int rowsTotal = STRIDED ? K : X, payload = STRIDED ? X : K;
    if (payload < E || K < E) return;
    const long long size = (long long)(rowsTotal - 1) * ld + payload;
    auto value = [&](long long e) { return (int)(e % 65521) + 1; };
    const int nk = (K + SMALL_STEP - 1) / SMALL_STEP;
    for (int x0 = 0; x0 < X; x0 += BX)
        for (int t = 0; t < nk; ++t) {
            const int k0 = t * SMALL_STEP, kLeft = K - k0, left = X - x0;
            const long long base = STRIDED ? (long long)k0 * ld + x0 : (long long)x0 * ld + k0;
            std::vector<int> stage(BX * SMALL_STEP, -1);
            for (int w = 0; w < NW; ++w)
                for (int lane = 0; lane < 64; ++lane)
                    for (int j = 0; j < small_chunks<BX, NW>(); ++j) {
                        int r = 0, c = 0, at = 0, sh = 0;
                        long long off = 0;
                        small_place<BX, NW, STRIDED>(j, w, lane, r, c, at);
                        if (t + 1 < nk) off = ragged_offset<STRIDED, E>(r, c, ld, left);
                        else ragged_last<STRIDED, E>(r, c, ld, left, kLeft, off, sh);
                        if (base + off < 0 || base + off + E > size) {
                            std::printf("strided %d X %d K %d ld %d x0 %d step %d: read %lld of %lld\n", STRIDED, X, K, ld, x0, t, base + off, size);
                            std::exit(1);
                        }
                        for (int e = 0; e < E; ++e) stage[at / 2 + e] = e + sh < E ? value(base + off + e + sh) : 0;
                    }
            // the fragments of the two 16-row blocks: 32 k each, eight to a step
            for (int block = 0; block < 2; ++block)
                for (int q = 0; q < 8; ++q)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int e = 0; e < E; ++e) {
                            const int x = block * 16 + (lane & 15), k = q * 32 + 8 * (lane >> 4) + e;
                            int at;
                            if constexpr (STRIDED) {
                                // lane i of a group of 16 receives column i of the block whose row i / 4 and columns 4 (i % 4) it addresses
                                const int i = lane & 15, src = (lane & ~15) | ((e & 3) * 4 + i / 4);
                                at = (b_frag_offset<BX>(block * 16, src, 0) + (e >> 2) * 4 * BX * 2 + q * (BX * 64)) / 2 + i % 4;
                            } else {
                                at = (a64_frag_offset(block * 16, lane, q & 1) + (q >> 1) * (BX * 128)) / 2 + e;
                            }
                            if (x0 + x >= X) continue;
                            const long long from = STRIDED ? (long long)(k0 + k) * ld + x0 + x : (long long)(x0 + x) * ld + k0 + k;
                            const int want = k0 + k < K ? value(from) : 0;
                            if (stage[at] != want) {
                                std::printf("strided %d X %d K %d ld %d: x %d k %d holds %d, not %d\n", STRIDED, X, K, ld, x0 + x, k0 + k, stage[at], want);
                                std::exit(1);
                            }
                            ++checked;
                        }
        }
}

int main()
{
    for (int X : {1, 7, 8, 9, 31, 32, 33, 40, 65, 100})
        for (int K : {8, 9, 31, 63, 64, 65, 255, 256, 257, 263, 264, 511, 512, 513, 769, 1031})
            for (int pad : {0, 1, 3, 8}) {
                run<false>(X, K, K + pad);
                run<true>(X, K, X + pad);
            }
    // tiles, slices of the plan, K, 64 x 64 tile of the plan, whether the kernel takes it
    struct { long long tiles; int slices, K; bool ragged, takes; } rule[] = {
        {60, 1, 640, true, true}, {256, 1, 8192, false, true}, {257, 1, 257, false, false}, {257, 1, 256, false, true}, {768, 1, 136, false, true},
        {769, 1, 136, false, false}, {512, 1, 128, false, true}, {513, 1, 128, false, false}, {257, 1, 64, false, false}, {256, 1, 64, false, true}, {1, 1, 8, false, true},
        {4, 1, 64, true, false}, {4, 1, 65, true, true}, {512, 1, 136, true, true}, {513, 1, 136, true, false}, {257, 1, 128, true, false},
        {72, 3, 1792, true, true}, {72, 3, 1793, true, false}, {72, 5, 2560, false, true}, {72, 5, 2568, false, false}, {257, 2, 2048, false, false}};
    for (auto &c : rule)
        if (small_tile_takes(c.tiles, c.slices, c.K, c.ragged) != c.takes) {
            std::printf("rule: %lld tiles, %d slices, K %d, ragged %d\n", c.tiles, c.slices, c.K, c.ragged);
            return 1;
        }
    if (small_run(1, 64) < 1 << 30 || small_run(3, 512) != 2 || small_run(3, 672) != 2 || small_run(8, 128) != 1) return 1;
    std::printf("small layout ok: %lld elements\n", checked);
    return 0;
}
