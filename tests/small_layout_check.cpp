// Host model of how the kernel of few output tiles fills its LDS stages and reads its fragments: every read lies inside the operand, every
// element of a step is where the fragment of its row and k is read, and which products take the kernel (test_gpu_small.py and test_gpu_f32_few.py lie on its sides).
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

// fp32: 32 x 32 tiles, or 16 x 16 ones whose waves share a step's k
template <int BT, bool STRIDED>
void run_f32(int X, int K, int ld)
{
    constexpr int STEP = few_step_f32(BT), PITCH = STRIDED ? few_pitch_b(BT) : few_pitch_a(BT), STAGE = STRIDED ? STEP * PITCH : BT * PITCH;
    const int rowsTotal = STRIDED ? K : X, payload = STRIDED ? X : K;
    if (payload < 4 || K < 4) return;
    const long long size = (long long)(rowsTotal - 1) * ld + payload;
    auto value = [&](long long e) { return (int)(e % 65521) + 1; };
    const int nk = (K + STEP - 1) / STEP;
    for (int x0 = 0; x0 < X; x0 += BT)
        for (int t = 0; t < nk; ++t) {
            const int k0 = t * STEP, left = X - x0;
            const long long base = STRIDED ? (long long)k0 * ld + x0 : (long long)x0 * ld + k0;
            std::vector<int> stage(STAGE / 4, -1);
            for (int w = 0; w < 4; ++w)
                for (int lane = 0; lane < 64; ++lane)
                    for (int j = 0; j < 4; ++j) {
                        int r = 0, c = 0, at = 0, sh = 0;
                        long long off = 0;
                        few_place_f32<BT, STRIDED>(j, w, lane, r, c, at);
                        if (t + 1 < nk) off = ragged_offset<STRIDED, 4>(r, c, ld, left);
                        else ragged_last<STRIDED, 4>(r, c, ld, left, K - k0, off, sh);
                        if (base + off < 0 || base + off + 4 > size || at % 16 || at + 16 > STAGE) {
                            std::printf("fp32 BT %d strided %d X %d K %d ld %d x0 %d step %d: read %lld of %lld, place %d\n", BT, STRIDED, X, K, ld, x0, t, base + off, size, at);
                            std::exit(1);
                        }
                        for (int e = 0; e < 4; ++e) stage[at / 4 + e] = e + sh < 4 ? value(base + off + e + sh) : 0;
                    }
            for (int x = 0; x < BT && x0 + x < X; ++x)
                for (int k = 0; k < STEP; ++k) {
                    const int at = (STRIDED ? few_at_b(BT, k, x) : few_at_a(BT, x, k)) / 4;
                    const long long from = STRIDED ? (long long)(k0 + k) * ld + x0 + x : (long long)(x0 + x) * ld + k0 + k;
                    const int want = k0 + k < K ? value(from) : 0;
                    if (stage[at] != want) {
                        std::printf("fp32 BT %d strided %d X %d K %d ld %d: x %d k %d holds %d, not %d\n", BT, STRIDED, X, K, ld, x0 + x, k0 + k, stage[at], want);
                        std::exit(1);
                    }
                    ++checked;
                }
        }
}

int main()
{
    for (int X : {1, 3, 4, 5, 15, 16, 17, 32, 33, 70})
        for (int K : {4, 5, 31, 127, 128, 129, 255, 256, 257, 515, 1023})
            for (int pad : {0, 1, 3}) {
                run_f32<32, false>(X, K, K + pad);
                run_f32<32, true>(X, K, X + pad);
                run_f32<16, false>(X, K, K + pad);
                run_f32<16, true>(X, K, X + pad);
            }
    struct { long long t16, t32; int K, tile; } few[] = {{256, 64, 256, 16}, {256, 64, 65, 16}, {256, 64, 64, 32}, {512, 140, 129, 16}, {512, 140, 128, 32}, {513, 140, 1000, 32},
                                                          {1024, 256, 64, 32}, {1100, 257, 256, 0}, {1100, 257, 257, 32}, {2048, 512, 512, 32}, {2052, 513, 512, 0}};
    for (auto &c : few)
        if (few_tile_f32(c.t16, c.t32, c.K) != c.tile) {
            std::printf("rule: %lld and %lld tiles, K %d\n", c.t16, c.t32, c.K);
            return 1;
        }
    for (int X : {1, 7, 8, 9, 31, 32, 33, 40, 65, 100})
        for (int K : {8, 9, 31, 63, 64, 65, 255, 256, 257, 263, 264, 511, 512, 513, 769, 1031})
            for (int pad : {0, 1, 3, 8}) {
                run<false>(X, K, K + pad);
                run<true>(X, K, X + pad);
            }
    // tiles, slices of the plan, K, 64 x 64 tile of the plan, whether the kernel takes it; and whether with rows that are slow to it, or with A stored K x M, where that differs
    struct { long long tiles; int slices, K; bool ragged, takes; int oddRows = -1, transA = -1; } rule[] = {
        {60, 1, 640, true, true}, {256, 1, 8192, false, true}, {257, 1, 257, false, false}, {257, 1, 256, false, true}, {768, 1, 136, false, true},
        {769, 1, 136, false, false}, {512, 1, 128, false, true}, {513, 1, 128, false, false}, {257, 1, 64, false, false}, {256, 1, 64, false, true}, {1, 1, 8, false, true},
        {4, 1, 64, true, false}, {4, 1, 65, true, true}, {512, 1, 136, true, true}, {513, 1, 136, true, false}, {257, 1, 128, true, false},
        {72, 3, 1536, true, true}, {72, 3, 1537, true, false}, {72, 4, 2552, false, true}, {65, 5, 2560, false, true, -1, 0}, {64, 5, 2560, false, false}, {193, 5, 2560, false, true}, {192, 5, 2560, false, true, -1, 0}, {4, 1, 256, true, true}, {4, 1, 257, true, true, 0}, {256, 1, 320, true, true, 0}, {4, 1, 321, true, true},
        {257, 1, 256, true, true}, {4, 1, 300, false, true}, {257, 2, 2048, false, false}};
    for (auto &c : rule)
        for (bool odd : {false, true})
            for (bool transA : {false, true})
                if (small_tile_takes(c.tiles, c.slices, c.K, c.ragged, transA, odd) != (odd && c.oddRows >= 0 ? c.oddRows != 0 : transA && c.transA >= 0 ? c.transA != 0 : c.takes)) {
                    std::printf("rule: %lld tiles, %d slices, K %d, ragged %d, odd rows %d, A K x M %d\n", c.tiles, c.slices, c.K, c.ragged, odd, transA);
                    return 1;
                }
    // rows at odd elements: M x K both (6), K x M A's (3, 7), with a residual both (15)
    for (int bits = 0; bits < 16; ++bits)
        if (small_odd_rows(bits & 1, bits & 2, bits & 4, bits & 8) != (bits == 3 || bits == 6 || bits == 7 || bits == 15)) return 1;
    struct { long long tiles; int slices, K; bool c8, takes; int bareF32 = -1; } conv[] = {{256, 1, 32, false, true}, {257, 1, 40, true, true, 0}, {512, 1, 32, false, true, 0}, {257, 1, 48, true, true},
        {768, 1, 128, false, true, 0}, {513, 1, 136, false, true}, {512, 1, 27 * 8, true, true}, {512, 1, 64, false, true}, {513, 1, 64, false, false}, {513, 1, 72, false, true, 0},
        {1024, 1, 136, false, true}, {1025, 1, 136, true, false}, {768, 1, 288, false, false}, {768, 1, 288, true, true}, {768, 1, 1152, false, true}, {769, 1, 1152, true, false},
        {512, 4, 2304, false, true}, {513, 4, 2304, false, false}, {20, 8, 4608, false, false}};
    for (auto &c : conv)
        for (bool bare : {false, true})
            if (small_conv_takes(c.tiles, c.slices, c.K, c.c8, bare) != (bare && c.bareF32 >= 0 ? c.bareF32 != 0 : c.takes)) {
                std::printf("rule of convolutions: %lld tiles, %d slices, K %d, c8 %d, bare fp32 %d\n", c.tiles, c.slices, c.K, c.c8, bare);
                return 1;
            }
    struct { bool plan128; long long blocks; int K; bool bf16; Tile64 kind, even = (Tile64)-1; } tiles[] = {{true, 1280, 64, false, TILE64_SHORT}, {true, 1281, 64, false, TILE64_SHORT, TILE64_NO}, {true, 4096, 64, false, TILE64_SHORT, TILE64_NO},
        {true, 256, 65, true, TILE64_RING}, {true, 256, 5000, false, TILE64_RING}, {true, 257, 65, false, TILE64_NO},
        {true, 768, 128, true, TILE64_RING}, {true, 257, 129, true, TILE64_NO}, {true, 769, 72, true, TILE64_NO}, {true, 1025, 72, true, TILE64_RING}, {true, 1537, 72, true, TILE64_NO},
        {false, 1280, 128, true, TILE64_RING}, {false, 1281, 72, true, TILE64_NO},
        {false, 100, 128, true, TILE64_NO}, {true, 768, 64, true, TILE64_SHORT}, {true, 769, 64, true, TILE64_SHORT_WIDE}, {true, 1024, 64, true, TILE64_SHORT_WIDE}, {false, 4096, 64, true, TILE64_SHORT}, {false, 4097, 64, true, TILE64_SHORT_WIDE}, {false, 4096, 64, false, TILE64_NO},
        {true, 256, 64, false, TILE64_SHORT}, {true, 257, 64, false, TILE64_NO}, {true, 1025, 64, false, TILE64_SHORT}, {true, 4097, 64, false, TILE64_NO}};
    for (auto &c : tiles)
        for (bool odd : {false, true})
            if (tile64_kind(c.plan128, c.blocks, c.K, c.bf16, odd) != (!odd && c.even != (Tile64)-1 ? c.even : c.kind)) {
                std::printf("rule of the 64 x 128 tile: %lld blocks, K %d, odd %d\n", c.blocks, c.K, odd);
                return 1;
            }
    for (bool odd : {false, true})
        if (conv_tile64_kind(true, 384, 1152, true, odd, true) != TILE64_RING || conv_tile64_kind(true, 384, 1160, true, odd, true) != TILE64_NO || conv_tile64_kind(true, 512, 576, true, odd, true) != TILE64_RING || conv_tile64_kind(true, 385, 584, true, odd, true) != TILE64_NO || conv_tile64_kind(true, 513, 264, true, odd, true) != TILE64_NO ||
            conv_tile64_kind(true, 768, 256, true, odd, true) != TILE64_RING || conv_tile64_kind(true, 257, 160, true, odd, false) != TILE64_NO || conv_tile64_kind(true, 256, 4608, false, odd, false) != TILE64_RING) {
            std::printf("rule of the 64 x 128 tile for convolutions\n");
            return 1;
        }
    if (small_run(1, 64) < 1 << 30 || small_run(3, 512) != 2 || small_run(3, 672) != 2 || small_run(8, 128) != 1) return 1;
    std::printf("small layout ok: %lld elements\n", checked);
    return 0;
}
