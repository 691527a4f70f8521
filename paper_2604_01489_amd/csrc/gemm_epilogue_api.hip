// C-ABI of the gfx950 fused GEMM library: argument validation, plan selection
// (direct / batched / split-K, tile shape) and kernel launches.  See
// include/gemm_epilogue.h for the contract of every entry point.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/gemm_epilogue.h"
#include "gemm_bf16_fast.h"
#include "gemm_bf16_w4.h"
#include "gemm_f32_fast.h"
#include "gemm_f32_few.h"
#include "gemm_f32_ragged.h"
#include "gemm_generic.h"
#include "gemm_ragged_launch.h"
#include "gemm_skinny.h"
#include "gemm_small_launch.h"
#include "gemm_tile64_launch.h"
#include "ge_host.h"
#include "plan_rates.h"
#include "small_layout.h"
#include "splitk_reduce.h"

namespace ge_host {

thread_local const char *g_last_config = "none";

thread_local hipError_t g_launch_error = hipSuccess;

// Library-owned buffers for partial results, one per (device, stream) that has needed one: calls on
// different streams never share a buffer, calls on one stream are ordered by it.
struct Workspace {
    int dev;
    hipStream_t stream;
    void *ptr;
    size_t bytes;
};
std::vector<Workspace> g_ws, g_ws_retired;
std::mutex g_ws_mutex;

// Switches for timing runs and tests: set by ge_set_option, initial values from the environment,
// read once when the library is loaded.
std::atomic<int> g_opt_force{FORCE_NONE};
std::atomic<int> g_opt_waves8{0}, g_opt_stage32{0}, g_opt_halo{HALO_AUTO};

int parse_force(const char *v)
{
    if (!v) return FORCE_NONE;
    if (std::strcmp(v, "256x256") == 0) return FORCE_256;
    if (std::strcmp(v, "128x128") == 0) return FORCE_128;
    if (std::strcmp(v, "generic") == 0) return FORCE_GENERIC;
    return -1;
}

int parse_halo(const char *v)
{
    if (!v) return HALO_AUTO;
    if (std::strcmp(v, "off") == 0) return HALO_OFF;
    if (std::strcmp(v, "on") == 0) return HALO_ON;
    if (std::strcmp(v, "14_11") == 0) return HALO_VARIANT0;
    if (std::strcmp(v, "12_12") == 0) return HALO_VARIANT0 + 1;
    return -1;
}

const bool g_env_read = [] {
    const int f = parse_force(std::getenv("GE_FORCE_CONFIG"));
    g_opt_force = f < 0 ? FORCE_NONE : f;
    const char *w = std::getenv("GE_WAVES"), *k = std::getenv("GE_STAGE_K");
    g_opt_waves8 = (w && std::strcmp(w, "8") == 0) ? 1 : 0;
    g_opt_stage32 = (k && std::strcmp(k, "32") == 0) ? 1 : 0;
    const int h = parse_halo(std::getenv("GE_CONV_HALO"));
    g_opt_halo = h < 0 ? HALO_AUTO : h;
    return true;
}();

int opt_force_config() { return g_opt_force.load(std::memory_order_relaxed); }
bool opt_eight_waves() { return g_opt_waves8.load(std::memory_order_relaxed) != 0; }
bool opt_stage_k32() { return g_opt_stage32.load(std::memory_order_relaxed) != 0; }
int opt_conv_halo() { return g_opt_halo.load(std::memory_order_relaxed); }

bool fast_path_ok(int N, int K, const void *A, int lda, const void *B, int ldb)
{
    if ((((uintptr_t)A) | ((uintptr_t)B)) & 15u) return false;
    if ((lda | ldb | N | K) & 7) return false;
    // per-lane byte offsets inside one tile panel must stay below 2^31
    if ((long long)lda * 2 * 256 + 256 >= (1ll << 31)) return false;
    if ((long long)ldb * 2 * 64 + 1024 >= (1ll << 31)) return false;
    return true;
}

// the tall-skinny kernel addresses a stage's 256 rows of B with 32-bit byte offsets
bool skinny_ld_ok(int ldb) { return (long long)ldb * 2 * 256 + 1024 < (1ll << 31); }

// K slices so that a launch with few output tiles still covers the chip (the guarded kernels; the
// direct-to-LDS kernels choose tile and slices together, see plan_cost_us).
int choose_split(long long tiles, int K, int minSlice)
{
    const int kMinSlice = minSlice;            // K extent below which a slice is not worth its partial tile
    if (tiles * 2 > kNumCU || K < 2 * kMinSlice) return 1;
    long long s = kNumCU / tiles;
    const long long maxS = K / kMinSlice;
    if (s > maxS) s = maxS;
    if (s > 64) s = 64;
    return s < 2 ? 1 : (int)s;
}

void slice_k(int K, int bk, int want, int *splitK, int *kPerSlice)
{
    int per = ceil_div(ceil_div(K, want), bk) * bk;
    if (per < bk) per = bk;
    *kPerSlice = per;
    *splitK = ceil_div(K, per);
}

// K slices of an fp32 product on tiles of `tile` squared that has to be sliced into at least `least` (a chain of sums over more of K is less
// exact): the count with the lowest estimate.  A CU's matrix pipes take 0.54 us for each 32-k step of each block it has been
// given (a 128 tile four times that), or a block alone 0.62 us with its waits; each round of blocks beyond the first begins and ends for
// 1.2 us (element by element, where a step takes several times as long, this does not count: 705 x 3 x 6400 22.6 with it, 20.9 without); the
// second pass is a launch, the partial tiles written and read and, for each slice, 0.057 us of round trips, eight slices each (without it 2 of 5 x 204 x 17484
// took 61 slices instead of 32: 20.4 us, 18.9 on these; 453 x 4 x 15976 63 instead of 31, 18.9 / 17.9).  What the count decides is how full the last round of blocks on the CUs
// is.  us, least / chosen: 1023 x 771 x 2049, 208 tiles, 4 slices 47.2 / 6 42.4 (5: 46.8, 7: 45.7); 320 x 320 x 4095, 7 19.2 / 10 16.4 (12:
// 20.6); 256 x 256 x 1024, 2 15.3 / 16 9.1 (8: 9.6); 72 x 1280 x 1600, 3 16.9 / 6 12.0.  Where the least count already
// is one round of the CUs, twice as many are no shorter: 80 x 966 x 4120, 8 19.4 (15: 20.5); 496 x 66 x 8368, 16 19.5 (30: 20.6); 2 of 460 x
// 40 x 8600, 16 18.9 (30: 19.9).  Slices keep 64 of K.
int f32_slices(int tile, long long tiles, long long outputs, int K, int least, bool elementwise)
{
    const double area = tile == 128 ? 4.0 : 1.0;
    int best = least;
    double bestCost = 0.0;
    for (int s = least; s <= 64 && (s == least || K / s >= 64); ++s) {
        const double rounds = (double)((tiles * s + kNumCU - 1) / kNumCU), steps = (double)ceil_div(ceil_div(K, s), 32);
        const double cost = steps * (rounds * area > 1.0 ? 0.54 * area * rounds : 0.62) + (elementwise ? 0.0 : 1.2 * (rounds - 1.0)) +
                            0.057 * s + (double)(s + 1) * (double)outputs * 4.0 / 4.5e6;
        if (s == least || cost < bestCost) { best = s; bestCost = cost; }
    }
    return best;
}

// Estimated time in microseconds of one structure -- block tile (256 or 128) and number of K slices --
// from a few measured rates (plan_rates.h, generated by the calibration run of tune.py): a launch of
// 256 x 256 blocks, one to a CU, takes kStep256Us per 32-wide K step plus kFixed256Us (the launch, the
// pipeline's fill, the tile's store), and every further round of blocks its steps plus kRound256Us; a
// 128 x 128 block has its own figures alone on a CU and others when two share it; K slices add the
// second pass (a launch and the partial tiles written and read).  Per output element the large tile is
// the cheaper one; the small one wins where the large one would leave CUs idle or need many slices.
// Checked against the timed search over both choices (tune.py): the rule is for ranking structures, not
// for predicting times.
double plan_cost_us(int M, int N, int K, int batch, int tile, int slices)
{
    const long long tiles = (long long)ceil_div(M, tile) * ceil_div(N, tile) * batch;
    const long long blocks = tiles * slices;
    const double steps = (double)ceil_div(ceil_div(K, slices), 32);
    double t;
    if (tile == 256) {
        const double rounds = (double)((blocks + kNumCU - 1) / kNumCU);
        t = steps * kStep256Us + kFixed256Us + (rounds - 1.0) * (steps * kStep256Us + kRound256Us);
    } else if (blocks <= kNumCU) {
        t = steps * kStep128AloneUs + kFixed128AloneUs;
    } else {
        const double rounds = (double)((blocks + 2 * kNumCU - 1) / (2 * kNumCU));
        t = steps * kStep128SharedUs + kFixed128SharedUs + (rounds - 1.0) * (steps * kStep128SharedUs + kRound128SharedUs);
    }
    if (slices > 1)
        t += kSecondPassLaunchUs + (double)(slices + 1) * (double)batch * (double)M * (double)N * 4.0 / kSecondPassBytesPerUs;
    return t;
}

// Multiply-adds above which the kernel for operands of any alignment takes what the direct-to-LDS kernels do not (us, guarded / any
// alignment: 130 x 70 x 1500, 13.7 M, 48.4 / 11.0; 513 x 515 x 33, 8.7 M, 7.5 / 5.2; 33 x 33 x 4096, 4.5 M, 27.7 / 8.4; 221 x 155 x
// 44, 1.5 M, 7.6 / 5.1), and products of aligned operands with few large tiles as well (small_tile_pays; 128 / 64 tile: 128 x 128 x 512 6.9 / 5.6,
// 200 x 200 x 400 7.4 / 5.3, 72 x 72 x 2040 22.1 / 12.7).  Not where the two cross: up to the line it is the shorter call too (128 x 128 x 64, on the line,
// 7.8 / 3.4; 100 x 100 x 100 10.4 / 4.5; 33 x 35 x 700 35.6 / 7.4; all of these on the 64 x 64 tile, from which gemm_small.h takes most), and so it is for K slices that the caller asks for up to kRaggedMinSliced; the
// configuration that these calls report is the guarded kernel's, which tests of that kernel count on.
constexpr double kRaggedMinWork = 1024.0 * 1024, kRaggedMinSliced = 16.0 * 1024 * 1024;

// The slice count of lowest estimated cost for a tile (1 = none); slices keep at least minSlice of K.
int best_slices(int M, int N, int K, int batch, int tile, int minSlice, double *cost)
{
    int best = 1;
    double bestCost = plan_cost_us(M, N, K, batch, tile, 1);
    // A product this short is over before a second launch has paid for itself: the rates are those of
    // a chip full of blocks, and a handful of blocks over K = 1024 take less than they predict (timed:
    // 128..1024 rows and columns at K = 1024 run 2-3 us faster in one pass, at K = 2048 slower).
    if (K < 2048) { if (cost) *cost = bestCost; return 1; }
    const int maxS = K / minSlice < 64 ? K / minSlice : 64;
    for (int s2 = 2; s2 <= maxS; ++s2) {
        const double c = plan_cost_us(M, N, K, batch, tile, s2);
        if (c < bestCost) { bestCost = c; best = s2; }
    }
    if (cost) *cost = bestCost;
    return best;
}

// Whether a product of aligned operands that takes no K slices is cheaper on the 64 x 64 tiles of the kernel for operands of
// any alignment (gemm_ragged.h): where the larger tiles leave CUs idle.  Its rates, us, from shapes of one to four blocks a
// CU: 5 for the launch, and per 64-k step 0.30 for a block alone on its CU or 0.22 for each that shares it.  The larger
// tiles' model is too dear where they do not fill the chip (1024^3: 15.9 modelled, 11.1 measured), hence the factor.  us,
// larger tile against this one: 1024^3 11.1 / 8.9; 1344 x 584 x 1712 20.3 / 12.2; 424 x 1024 x 1920 (B N x K, bf16 out) 17.2 /
// 11.8; 39 x 4160 x 1128 13.7 / 10.0; left alone: 1536^3 16.4 / 20.1; 640 x 5616 x 448 9.0 / 11.9; 1384 x 1024 x 1664 16.6 /
// 16.3; with slices on both 512 x 512 x 4096 14.7 / 15.2.
bool small_tile_pays(int M, int N, int K, int batch, double otherCost)
{
    const long long tiles = (long long)ceil_div(M, 64) * ceil_div(N, 64) * batch;
    const double share = (double)((tiles + kNumCU - 1) / kNumCU), steps = (double)ceil_div(K, 64);
    return 5.0 + steps * (0.22 * share > 0.30 ? 0.22 * share : 0.30) < 0.7 * otherCost;
}
// Products shorter than this stay on the larger tiles: there both are a launch and little else, and the line is not where they
// cross (us, 128 tile / this one: 736 x 320 x 320 5.8 / 5.0, 512 x 512 x 256 5.4 / 5.0, 1024 x 512 x 352 6.1 / 5.4, 520 x 776 x 128
// 5.1 / 4.8; above the line 1024 x 1024 x 1024 11.1 / 8.9).  Of these the line decides little by now: where they are few tiles the 32 x 32 or the 64 x 128 one takes them from whichever
// plan they have (512 x 512 x 256, 1024 x 512 x 352).
constexpr int kSmallTileMinK = 384;

bool ragged_ok(int M, int N, int K, int batch, int lda, bool transA, int ldb, bool transB, int ldc, bool plain)
{
    if (ldc >= ge::EDGE_LDC_MAX) return false;
    if (opt_force_config() == FORCE_GENERIC) return false;
    // the last step pulls a chunk that hangs over the end of its row back inside the row
    if (K < 8 || (transA && M < 8) || (!transB && N < 8)) return false;
    // byte offsets of a lane inside a tile panel: 128 rows along k, or 64 rows along M or N
    if ((long long)lda * (transA ? 128 : 256) + 1024 >= (1ll << 31) || (long long)ldb * (transB ? 256 : 128) + 1024 >= (1ll << 31)) return false;
    // Slivers of the plain operator, of whose 64 x 64 tiles there are four or more to a CU with one output in ten or fewer inside, and one 32-k
    // step or, in few multiply-adds, a few k past a 64-k step: the guarded kernel reads no more than is there.  us, guarded / any alignment: 2 x 185 x 9, 3794 of
    // them, 28.2 / 34.0; 6 x 10 x 9, 3568, 10.7 / 12.4; 1 x 567 x 16, 227, 7.5 / 8.2; 6 x 3596 x 23, 20, 5.7 / 6.5; 2 x 734 x 68, 100, 7.8 / 10.5; 3 x 3906 x
    // 65, 20, 8.1 / 9.4; 5 x 350 x 28, 500, 11.0 / 20.9; the other side: 4 x 4426 x 66, 100, 55.0 / 28.6; 1 x 4932 x 65, 100, 56.4 / 40.3; 18 x 37 x 12, 1273, 7.3 / 6.9; 2 x 55 x 14, 741, 4.9 / 4.8; 1 x 209 x 40, 500, 9.5 / 8.1; 4 x 69 x 57, 500, 6.7 / 5.0;
    // with the widened operator's chain 1 x 237 x 19, 1562, 31.4 / 19.9.
    const double tiles = (double)ceil_div(M, 64) * ceil_div(N, 64) * batch;
    const double work = (double)M * N * K * batch;
    if (plain && (K <= 32 || (K > 64 && K <= 72 && work < 16.0 * 1024 * 1024)) && tiles >= 4.0 * kNumCU && 10.0 * M * N * batch <= 4096.0 * tiles) return false;
    return work > kRaggedMinWork;
}

ge_status_t make_plan_bf16(int M, int N, int K, int batch, bool fast, ge_plan_t plan, int split_k, Plan *out, bool skinny, bool ragged)
{
    Plan pl{};
    if (plan != GE_PLAN_AUTO && plan != GE_PLAN_DIRECT && plan != GE_PLAN_SPLITK) return GE_ERR_CONFIG;
    if (split_k < 0) return GE_ERR_CONFIG;
    const int force = opt_force_config();
    int want = 1;
    if (skinny && fast && force == FORCE_NONE && N <= 32 && M >= 1024 && batch <= 65535) {
        // Many rows, at most 32 columns: a stream of A.  32 rows and every column per workgroup; K is
        // sliced only where the rows alone do not make enough workgroups, into slices of 1024 or more.
        pl.tile = TILE_SKINNY; pl.bm = 32; pl.bn = N <= 16 ? 16 : 32; pl.bk = ge_skinny::KS;
        const long long blocks = (long long)ceil_div(M, 32) * batch;
        int autoS = 1;
        if (blocks < 192) {
            autoS = (int)((kNumCU + blocks - 1) / blocks);
            if (autoS > K / 1024) autoS = K / 1024;
            if (autoS < 1) autoS = 1;
        }
        if (plan == GE_PLAN_DIRECT) want = 1;
        else if (plan == GE_PLAN_SPLITK) want = split_k > 0 ? (split_k < 2 ? 2 : split_k) : (autoS < 2 ? 2 : autoS);
        else want = autoS;
    } else if (!fast || force == FORCE_GENERIC) {
        pl.tile = TILE_GENERIC; pl.bm = 64; pl.bn = 64; pl.bk = 32;
        const long long tiles = (long long)ceil_div(M, 64) * ceil_div(N, 64) * batch;
        if (plan == GE_PLAN_SPLITK) want = split_k > 0 ? split_k : choose_split(tiles, K, 512);
        else if (plan == GE_PLAN_AUTO) want = choose_split(tiles, K, 512);
        if (plan == GE_PLAN_SPLITK && want < 2) want = 2;
        if (ragged && force != FORCE_GENERIC && (plan != GE_PLAN_SPLITK || (double)M * N * K * batch >= kRaggedMinSliced)) {
            // the same slices on the larger tiles of gemm_ragged.h: 128 x 128 where they make three blocks for every
            // four CUs, else 64 x 64 (64 against 128, us: 1999 x 1537 x 2051, 208 blocks of 128, 45 / 34; 3001 x 3001 x
            // 901, 576 blocks, 47 / 42; 1031 x 2051 x 1024, 153 blocks, 17.1 / 17.3; 1001^3, 64 blocks, 9.4 / 19.5), and where
            // such a tile takes the place of two and a half small ones or more, else much of it is padding (two: batches of 16, K = 48,
            // 9 x 4099 8.7 / 12.2, 48 x 2316 8.2 / 10.6; 48 x 30001 x 2049 25.7 / 28.5; 2.25: 300 of 129 x 129 x 33 16.2 / 20.8, x 1025
            // 63 / 76; 2.5: 40 of 129 x 300 x 65 7.7 / 7.8, x 2049 43 / 37; 3.3: 200 of 67 x 300 x 48 16.7 / 15.5).  Fewer of the large
            // ones, but more than two small ones to a CU, and K long enough for what the second round of these costs: the
            // large ones too (1601^3 31.6 / 27.2, 1501 x 1501 x 2051 35.8 / 30.0, 1405 x 1501 x 1501, 528 small ones, 29.1 / 25.2, 40 of 200 x
            // 200 x 1001 19.2 / 16.5; two or fewer: 1401^3, 484, 19.1 / 22.7, 901 x 2049 x 1024, 495, 14.2 / 17.2, 25 of 129 x 300 x
            // 2049, 375, 23.9 / 27.5; short K: 1405 x 1501 x 301 10.2 / 10.3, 1700 x 1700 x 129 8.6 / 9.1, 1601 x 1601 x 33 7.3 / 8.2)
            const long long t128 = (long long)ceil_div(M, 128) * ceil_div(N, 128) * batch;
            const bool fills = t128 * want * 4 >= kNumCU * 3 || (tiles * want > 2 * kNumCU && K / want > 256);
            const bool big = fills && 2 * tiles >= 5 * t128;
            pl.tile = big ? TILE_RAGGED_128 : TILE_RAGGED_64;
            pl.bm = pl.bn = big ? 128 : 64;
            pl.bk = 64;
        }
    } else {
        // both tiles are candidates when the problem has 256 rows and columns; each with the slice
        // count the plan asks for (none, the caller's, or its own best), the cheaper structure wins
        constexpr int kMinSlice = 512;
        int tileOf[2] = {256, 128}, slicesOf[2] = {1, 1};
        double costOf[2] = {0.0, 0.0};
        for (int c = 0; c < 2; ++c) {
            if (plan == GE_PLAN_DIRECT) slicesOf[c] = 1;
            else if (plan == GE_PLAN_SPLITK && split_k > 0) slicesOf[c] = split_k < 2 ? 2 : split_k;
            else {
                slicesOf[c] = best_slices(M, N, K, batch, tileOf[c], kMinSlice, nullptr);
                if (plan == GE_PLAN_SPLITK && slicesOf[c] < 2) slicesOf[c] = 2;
            }
            costOf[c] = plan_cost_us(M, N, K, batch, tileOf[c], slicesOf[c]);
        }
        bool big = (M >= 256 && N >= 256) && costOf[0] <= costOf[1];
        if (force == FORCE_256) big = true;
        if (force == FORCE_128) big = false;
        const int chosen = big ? 0 : 1;
        if (ragged && force == FORCE_NONE && plan == GE_PLAN_AUTO && K >= kSmallTileMinK && slicesOf[chosen] == 1 &&
            small_tile_pays(M, N, K, batch, costOf[chosen])) { pl.tile = TILE_RAGGED_64; pl.bm = pl.bn = 64; pl.bk = 64; }
        else if (big) { pl.tile = TILE_256; pl.bm = 256; pl.bn = 256; pl.bk = ge::BF16_BK; want = slicesOf[0]; }
        else     { pl.tile = TILE_128; pl.bm = 128; pl.bn = 128; pl.bk = ge::BF16_BK; want = slicesOf[1]; }
    }
    pl.tilesM = ceil_div(M, pl.bm);
    pl.tilesN = ceil_div(N, pl.bn);
    const long long tiles = (long long)pl.tilesM * pl.tilesN * batch;
    // (operands of any alignment: the guarded kernel's 64 x 64 tiles set the limit, whichever tile they get)
    const long long counted = pl.tile == TILE_RAGGED_128 ? (long long)ceil_div(M, 64) * ceil_div(N, 64) * batch : tiles;
    if (counted > 0x7fffffffll / 64) return GE_ERR_SHAPE;
    // (a block of the kernel for any alignment ends anywhere in a step: its slices are the guarded kernel's)
    const bool anyAlignment = pl.tile == TILE_RAGGED_128 || pl.tile == TILE_RAGGED_64;
    slice_k(K, anyAlignment ? 32 : pl.bk, want, &pl.splitK, &pl.kPerSlice);
    if (pl.splitK == 1) pl.kPerSlice = ceil_div(K, pl.bk) * pl.bk;
    if (counted * pl.splitK > 0x7fffffffll) return GE_ERR_SHAPE;
    pl.edgeMN = (M % pl.bm) || (N % pl.bn);
    pl.edge = (M % pl.bm) || (N % pl.bn) || (K % pl.bk) || (pl.kPerSlice % pl.bk);
    if (pl.tile == TILE_SKINNY) {
        pl.tilesN = 1;
        if ((long long)pl.tilesM * pl.splitK > 0x7fffffffll) return GE_ERR_SHAPE;
    }
    *out = pl;
    return GE_OK;
}

ge_status_t make_plan_bf16_for(int M, int N, int K, int batch, bool fast, ge_plan_t plan, int split_k, int ldc, bool f32Out, Plan *out, bool skinny,
                               bool ragged)
{
    ge_status_t st = make_plan_bf16(M, N, K, batch, fast, plan, split_k, out, skinny, ragged);
    if (st != GE_OK || !out->edgeMN || (out->tile != TILE_256 && out->tile != TILE_128)) return st;
    const int rowLength = out->splitK > 1 ? N : f32Out ? ldc : 0;      // of what is stored through 31-bit offsets
    return rowLength < ge::EDGE_LDC_MAX ? st : make_plan_bf16(M, N, K, batch, false, plan, split_k, out);
}

bool small_ok(const Plan &pl, const GemmParams &p, ge_plan_t plan)
{
    if ((pl.tile != TILE_128 && pl.tile != TILE_RAGGED_64) || p.triA != ge::TRI_NONE || plan == GE_PLAN_SPLITK || opt_force_config() != FORCE_NONE) return false;
    // 256 rows along k, or 32 along M or N
    if ((long long)p.lda * (p.transA ? 512 : 64) + 1024 >= (1ll << 31) || (long long)p.ldb * (p.transB ? 64 : 512) + 1024 >= (1ll << 31)) return false;
    const bool oddA = ((uintptr_t)p.A & 2u) != 0 || (p.lda & 1), oddB = ((uintptr_t)p.B & 2u) != 0 || (p.ldb & 1);
    return ge::small_tile_takes((long long)ceil_div(p.M, 32) * ceil_div(p.N, 32) * p.batch, pl.splitK, p.K, pl.tile == TILE_RAGGED_64, p.transA != 0,
                                p.cType == ge::DT_F32 && ge::small_odd_rows(p.transA != 0, oddA, oddB, p.R != nullptr));
}

size_t partial_bytes(int M, int N, int batch, int splitK)
{
    return splitK <= 1 ? 0 : (size_t)splitK * (size_t)batch * (size_t)M * (size_t)N * sizeof(float);
}

ge_status_t validate(int M, int N, int K, const void *A, int lda, const void *B, int ldb,
                     const void *bias, int act, const void *C, int ldc, int batch, size_t elem)
{
    if (!A || !B || !C) return GE_ERR_NULL;
    if (M < 1 || N < 1 || K < 1 || batch < 1) return GE_ERR_SHAPE;
    if (lda < K || ldb < N || ldc < N) return GE_ERR_LD;
    if (act != GE_ACT_NONE && act != GE_ACT_RELU && act != GE_ACT_GELU_TANH) return GE_ERR_ACT;
    if (((uintptr_t)A % elem) || ((uintptr_t)B % elem) || ((uintptr_t)C % 4) || ((uintptr_t)bias % 4))
        return GE_ERR_ALIGN;
    // element counts of one operand must fit 63 bits comfortably
    const long double big = 9.0e18L;
    if ((long double)batch * M * lda > big || (long double)batch * K * ldb > big ||
        (long double)batch * M * ldc > big)
        return GE_ERR_SHAPE;
    return GE_OK;
}

GemmParams base_params(int M, int N, int K, const void *A, int lda, const void *B, int ldb,
                       const float *bias, float alpha, int act, float *C, int ldc, int batch)
{
    GemmParams p{};
    p.A = A; p.B = B; p.bias = bias; p.C = C;
    p.M = M; p.N = N; p.K = K;
    p.lda = lda; p.ldb = ldb; p.ldc = ldc;
    p.strideA = (long long)M * lda;
    p.strideB = (long long)K * ldb;
    p.strideC = (long long)M * ldc;
    p.sliceStride = (long long)batch * M * N;
    p.batch = batch;
    p.splitK = 1;
    p.alpha = alpha;
    p.act = act;
    p.bytesA = 0;
    p.bytesB = 0;
    return p;
}

// Tile rows swept together: enough that the ~32 tiles resident on one XCD form
// a compact block (A panels and B panels both reused from that XCD's L2).
int choose_group_m(int tilesM, int tilesN)
{
    int g = 8;
    if (tilesN < 4) g = 32 / (tilesN < 1 ? 1 : tilesN);
    if (g > tilesM) g = tilesM;
    return g < 1 ? 1 : g;
}

ge_status_t acquire_workspace(size_t need, void *user, size_t user_bytes, hipStream_t stream, void **out)
{
    if (user) {
        if (user_bytes < need || ((uintptr_t)user & 255u)) return GE_ERR_WORKSPACE;
        *out = user;
        return GE_OK;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return GE_ERR_WORKSPACE;
    std::lock_guard<std::mutex> lock(g_ws_mutex);
    Workspace *ws = nullptr;
    for (Workspace &w : g_ws)
        if (w.dev == dev && w.stream == stream) { ws = &w; break; }
    if (ws && ws->bytes >= need) {
        *out = ws->ptr;
        return GE_OK;
    }
    // A larger buffer is needed.  hipMalloc is not a capturable operation, and a graph captured
    // now would keep replaying into whatever address it recorded: refuse instead.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return GE_ERR_WORKSPACE;
    void *ptr = nullptr;
    if (hipMalloc(&ptr, need) != hipSuccess) return GE_ERR_WORKSPACE;
    if (ws) {
        // work enqueued earlier (or a graph captured earlier) may still use the outgrown buffer
        g_ws_retired.push_back(Workspace{dev, nullptr, ws->ptr, 0});
        ws->ptr = ptr;
        ws->bytes = need;
    } else {
        g_ws.push_back(Workspace{dev, stream, ptr, need});
    }
    *out = ptr;
    return GE_OK;
}

ge_status_t reserve_workspace(size_t need, void *user, size_t user_bytes, hipStream_t stream)
{
    void *unused = nullptr;
    if (need == 0 || acquire_workspace(need, user, user_bytes, stream, &unused) == GE_OK) return GE_OK;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    return !user && hipStreamIsCapturing(stream, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone ? GE_OK : GE_ERR_WORKSPACE;
}

template <int EDGE>
hipError_t launch_four_wave(const GemmParams &p, bool raw, int act, dim3 grid, hipStream_t st)
{
    if (raw) {
        GE_LAUNCH((ge::gemm_bf16_w4_kernel<EDGE, true, ge::ACT_NONE, false, false, false, false>), grid, dim3(256), 0, st, p);
    } else if (act == GE_ACT_RELU) {
        GE_LAUNCH((ge::gemm_bf16_w4_kernel<EDGE, false, ge::ACT_RELU, false, false, false, false>), grid, dim3(256), 0, st, p);
    } else if (act == GE_ACT_GELU_TANH) {
        GE_LAUNCH((ge::gemm_bf16_w4_kernel<EDGE, false, ge::ACT_GELU_TANH, false, false, false, false>), grid, dim3(256), 0, st, p);
    } else {
        GE_LAUNCH((ge::gemm_bf16_w4_kernel<EDGE, false, ge::ACT_NONE, false, false, false, false>), grid, dim3(256), 0, st, p);
    }
    return ge_host::take_launch_error();
}

template <int BM, int BN, int WM, int WN, int EDGE>
hipError_t launch_fast_sel(const GemmParams &p, bool raw, int act, dim3 grid, hipStream_t st)
{
    constexpr int threads = WM * WN * 64;
    if (raw) {
        GE_LAUNCH((ge::gemm_bf16_kernel<BM, BN, WM, WN, EDGE, true, ge::ACT_NONE>), grid, dim3(threads), 0, st, p);
    } else if (act == GE_ACT_RELU) {
        GE_LAUNCH((ge::gemm_bf16_kernel<BM, BN, WM, WN, EDGE, false, ge::ACT_RELU>), grid, dim3(threads), 0, st, p);
    } else if (act == GE_ACT_GELU_TANH) {
        GE_LAUNCH((ge::gemm_bf16_kernel<BM, BN, WM, WN, EDGE, false, ge::ACT_GELU_TANH>), grid, dim3(threads), 0, st, p);
    } else {
        GE_LAUNCH((ge::gemm_bf16_kernel<BM, BN, WM, WN, EDGE, false, ge::ACT_NONE>), grid, dim3(threads), 0, st, p);
    }
    return ge_host::take_launch_error();
}

template <int BM, int BN, int WM, int WN>
hipError_t launch_fast(const GemmParams &p, int edge, bool raw, int act, dim3 grid, hipStream_t st)
{
    if (edge == 2) return launch_fast_sel<BM, BN, WM, WN, 2>(p, raw, act, grid, st);
    if (edge == 1) return launch_fast_sel<BM, BN, WM, WN, 1>(p, raw, act, grid, st);
    return launch_fast_sel<BM, BN, WM, WN, 0>(p, raw, act, grid, st);
}

hipError_t launch_reduce(const GemmParams &p, const void *ws, bool plain, hipStream_t st)
{
    // four outputs a lane where that still gives every CU a block (8192 x 8 over 32 terms: 27.9 us the call with four, 27.4 with one)
    const int vec = p.N % 4 == 0 && (double)p.batch * p.M * p.N >= 4.0 * 256 * kNumCU ? 4 : 1, pieces = ceil_div(p.N, vec);
    int lg = 0;
    while (lg < 6 && (1 << lg) < pieces) ++lg;
    const long long rowBlocks = ((long long)p.batch * p.M + (256 >> lg) - 1) / (256 >> lg);
    const dim3 grid((unsigned)ceil_div(pieces, 1 << lg), (unsigned)(rowBlocks < 65535 ? rowBlocks : 65535));
    const float *W = (const float *)ws;
    if (plain) {
        if (vec == 4) GE_LAUNCH((ge::splitk_reduce_kernel<true, 4>), grid, dim3(256), 0, st, p, W, lg);
        else          GE_LAUNCH((ge::splitk_reduce_kernel<true, 1>), grid, dim3(256), 0, st, p, W, lg);
    } else {
        if (vec == 4) GE_LAUNCH((ge::splitk_reduce_kernel<false, 4>), grid, dim3(256), 0, st, p, W, lg);
        else          GE_LAUNCH((ge::splitk_reduce_kernel<false, 1>), grid, dim3(256), 0, st, p, W, lg);
    }
    return ge_host::take_launch_error();
}

bool four_wave_ok(const Plan &pl, int K)
{
    if (opt_eight_waves()) return false;
    const int range = pl.splitK > 1 ? pl.kPerSlice : K;
    return pl.tile == TILE_256 && range >= 256;
}

int four_wave_edge(const Plan &pl, int K)
{
    if (K % 128 != 0 || (pl.splitK > 1 && pl.kPerSlice % 128 != 0)) return 2;
    return pl.edge ? 1 : 0;
}

int tile_edge(const Plan &pl, int K, int step)
{
    if (K % step != 0 || (pl.splitK > 1 && pl.kPerSlice % step != 0)) return 2;
    return pl.edgeMN ? 1 : 0;
}

ge_status_t run_bf16(int M, int N, int K, const uint16_t *A, int lda, const uint16_t *B, int ldb,
                     const float *bias, float alpha, ge_act_t act, float *C, int ldc, int batch,
                     ge_plan_t plan, int split_k, void *workspace, size_t workspace_bytes, void *stream)
{
    ge_status_t st = validate(M, N, K, A, lda, B, ldb, bias, (int)act, C, ldc, batch, 2);
    if (st != GE_OK) return st;
    Plan pl;
    st = make_plan_bf16_for(M, N, K, batch, fast_path_ok(N, K, A, lda, B, ldb), plan, split_k, ldc, true, &pl, skinny_ld_ok(ldb),
                            ragged_ok(M, N, K, batch, lda, false, ldb, false, ldc, true));
    if (st != GE_OK) return st;

    GemmParams p = base_params(M, N, K, A, lda, B, ldb, bias, alpha, (int)act, C, ldc, batch);
    p.tilesM = pl.tilesM;
    p.tilesN = pl.tilesN;
    p.groupM = choose_group_m(pl.tilesM, pl.tilesN);
    p.splitK = pl.splitK;
    p.kPerSlice = pl.kPerSlice;

    // extent of the operands as the arguments describe them (last row ends at its last element)
    p.bytesA = 2 * (((long long)batch * M - 1) * lda + K);
    p.bytesB = 2 * (((long long)batch * K - 1) * ldb + N);

    const bool sliced = pl.splitK > 1, small = small_ok(pl, p, plan), raw = sliced && !small;
    const Tile64 tile64 = small ? TILE64_NO : tile64_of(pl, p, plan);
    if (small || tile64 != TILE64_NO) {          // the run-time consumer chain, with nothing beyond the plain operator's
        p.clampLo = -INFINITY;
        p.clampHi = INFINITY;
    }
    void *ws = nullptr;
    if (small) {
        st = reserve_workspace(partial_bytes(M, N, batch, pl.splitK), workspace, workspace_bytes, (hipStream_t)stream);
        if (st != GE_OK) return st;
    }
    if (raw) {
        st = acquire_workspace(partial_bytes(M, N, batch, pl.splitK), workspace, workspace_bytes, (hipStream_t)stream, &ws);
        if (st != GE_OK) return st;
        p.C = (float *)ws;
    }
    const dim3 grid((unsigned)((long long)pl.tilesM * pl.tilesN * batch * pl.splitK));
    hipStream_t hs = (hipStream_t)stream;
    hipError_t err;
    if (small || tile64 != TILE64_NO) {
        if (small) launch_small(p, hs);
        else       launch_tile64(p, tile64, hs);
        g_last_config = small ? "bf16_small_32x32x256" : tile64_config(tile64, TILE64_PLAIN);
        return ge_host::take_launch_error() != hipSuccess ? GE_ERR_LAUNCH : GE_OK;
    }
    switch (pl.tile) {
    case TILE_SKINNY: {
        const dim3 sgrid((unsigned)((long long)pl.tilesM * pl.splitK), (unsigned)batch);
        // many workgroups: a ring of four stages, so that two or three share a CU; about one to a CU: eight
        const bool deep = (long long)sgrid.x * sgrid.y < 2 * kNumCU;
        auto launch = [&](auto np, auto rawC) {
            constexpr int NP = decltype(np)::value;
            constexpr bool R = decltype(rawC)::value;
            if (deep) GE_LAUNCH((ge::gemm_skinny_bf16_kernel<NP, R, 8>), sgrid, dim3(256), 0, hs, p);
            else      GE_LAUNCH((ge::gemm_skinny_bf16_kernel<NP, R, 4>), sgrid, dim3(256), 0, hs, p);
        };
        if (pl.bn == 16) {
            if (raw) launch(std::integral_constant<int, 16>{}, std::true_type{});
            else     launch(std::integral_constant<int, 16>{}, std::false_type{});
        } else {
            if (raw) launch(std::integral_constant<int, 32>{}, std::true_type{});
            else     launch(std::integral_constant<int, 32>{}, std::false_type{});
        }
        err = ge_host::take_launch_error();
        g_last_config = raw ? "bf16_skinny_32xN_k128_splitk" : "bf16_skinny_32xN_k128";
        break;
    }
    case TILE_256:
        if (four_wave_ok(pl, K)) {
            const int mode = four_wave_edge(pl, K);
            err = mode == 2 ? launch_four_wave<2>(p, raw, (int)act, grid, hs)
                : mode == 1 ? launch_four_wave<1>(p, raw, (int)act, grid, hs) : launch_four_wave<0>(p, raw, (int)act, grid, hs);
            g_last_config = raw ? "bf16_256x256x64_w4_splitk" : "bf16_256x256x64_w4";
            break;
        }
        err = launch_fast<256, 256, 2, 4>(p, tile_edge(pl, K, 32), raw, (int)act, grid, hs);
        g_last_config = raw ? "bf16_256x256x32_w8_splitk" : "bf16_256x256x32_w8";
        break;
    case TILE_128:
        err = launch_fast<128, 128, 2, 2>(p, tile_edge(pl, K, 32), raw, (int)act, grid, hs);
        g_last_config = raw ? "bf16_128x128x32_w4_splitk" : "bf16_128x128x32_w4";
        break;
    case TILE_RAGGED_128:
    case TILE_RAGGED_64:
        p.clampLo = -INFINITY;       // the run-time consumer chain, with nothing beyond the plain operator's
        p.clampHi = INFINITY;
        if (pl.tile == TILE_RAGGED_128) launch_ragged_128(p, raw, grid, hs);
        else                            launch_ragged_64(p, raw, grid, hs);
        err = ge_host::take_launch_error();
        g_last_config = pl.tile == TILE_RAGGED_128 ? (raw ? "bf16_ragged_128x128x64_splitk" : "bf16_ragged_128x128x64")
                                                   : (raw ? "bf16_ragged_64x64x64_splitk" : "bf16_ragged_64x64x64");
        break;
    default:
        if (raw) GE_LAUNCH(ge::gemm_bf16_generic_kernel<true>, grid, dim3(256), 0, hs, p);
        else     GE_LAUNCH(ge::gemm_bf16_generic_kernel<false>, grid, dim3(256), 0, hs, p);
        err = ge_host::take_launch_error();
        g_last_config = raw ? "bf16_generic_64x64x32_splitk" : "bf16_generic_64x64x32";
        break;
    }
    if (err != hipSuccess) return GE_ERR_LAUNCH;
    if (raw) {
        p.C = C;
        err = launch_reduce(p, ws, true, hs);
        if (err != hipSuccess) return GE_ERR_LAUNCH;
    }
    return GE_OK;
}

// ---- scratch for the entry point that allocates nothing -----------------------------------------
// Partial tiles of gemm_epilogue_bf16_static live in this array, which every GPU the library runs
// on holds, at its own address, until the process ends.  In host code the array's name is not a
// device address: the address is asked for once per device (with that device current) and kept.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
constexpr int kMaxDevices = 64;
void *g_static_scratch_ptr[kMaxDevices] = {};
std::mutex g_static_scratch_mutex;

}  // namespace ge_host

static __device__ __align__(256) unsigned char scratch[ge_host::kStaticScratchBytes];

namespace ge_host {

ge_status_t static_scratch(void **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GE_ERR_WORKSPACE;
    std::lock_guard<std::mutex> lock(g_static_scratch_mutex);
    if (!g_static_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return GE_ERR_WORKSPACE;
        g_static_scratch_ptr[dev] = ptr;
    }
    *out = g_static_scratch_ptr[dev];
    return GE_OK;
}

}  // namespace ge_host

using namespace ge_host;

extern "C" {

ge_status_t gemm_epilogue_bf16(int M, int N, int K, const uint16_t *A, int lda, const uint16_t *B, int ldb,
                               const float *bias, float alpha, ge_act_t act, float *C, int ldc,
                               int batch, void *stream)
{
    return run_bf16(M, N, K, A, lda, B, ldb, bias, alpha, act, C, ldc, batch, GE_PLAN_AUTO, 0, nullptr, 0, stream);
}

ge_status_t gemm_epilogue_bf16_ex(int M, int N, int K, const uint16_t *A, int lda, const uint16_t *B, int ldb,
                                  const float *bias, float alpha, ge_act_t act, float *C, int ldc,
                                  int batch, ge_plan_t plan, int split_k, void *workspace,
                                  size_t workspace_bytes, void *stream)
{
    return run_bf16(M, N, K, A, lda, B, ldb, bias, alpha, act, C, ldc, batch, plan, split_k, workspace,
                    workspace_bytes, stream);
}

ge_status_t gemm_epilogue_bf16_static(int M, int N, int K, const uint16_t *A, int lda, const uint16_t *B, int ldb,
                                      const float *bias, float alpha, ge_act_t act, float *C, int ldc,
                                      int batch, ge_plan_t plan, int split_k, void *stream)
{
    ge_status_t st = validate(M, N, K, A, lda, B, ldb, bias, (int)act, C, ldc, batch, 2);
    if (st != GE_OK) return st;
    Plan pl;
    st = make_plan_bf16_for(M, N, K, batch, fast_path_ok(N, K, A, lda, B, ldb), plan, split_k, ldc, true, &pl, skinny_ld_ok(ldb),
                            ragged_ok(M, N, K, batch, lda, false, ldb, false, ldc, true));
    if (st != GE_OK) return st;
    void *ws = nullptr;
    if (pl.splitK > 1) {
        if (partial_bytes(M, N, batch, pl.splitK) > kStaticScratchBytes) return GE_ERR_WORKSPACE;
        st = static_scratch(&ws);
        if (st != GE_OK) return st;
    }
    // with a workspace in hand the common path neither allocates nor frees; every partial tile is
    // written before the second pass reads it, so what an earlier call left in the array is never seen
    return run_bf16(M, N, K, A, lda, B, ldb, bias, alpha, act, C, ldc, batch, plan, split_k, ws,
                    ws ? kStaticScratchBytes : 0, stream);
}

size_t gemm_epilogue_static_scratch_bytes(void) { return kStaticScratchBytes; }

ge_status_t gemm_epilogue_f32(int M, int N, int K, const float *A, int lda, const float *B, int ldb,
                              const float *bias, float alpha, ge_act_t act, float *C, int ldc,
                              int batch, void *stream)
{
    ge_status_t st = validate(M, N, K, A, lda, B, ldb, bias, (int)act, C, ldc, batch, 4);
    if (st != GE_OK) return st;
    GemmParams p = base_params(M, N, K, A, lda, B, ldb, bias, alpha, (int)act, C, ldc, batch);
    p.bytesA = 4 * (((long long)batch * M - 1) * lda + K);
    p.bytesB = 4 * (((long long)batch * K - 1) * ldb + N);
    p.splitK = 1;
    p.kPerSlice = ceil_div(K, 16) * 16;
    hipStream_t hs = (hipStream_t)stream;
    // direct-to-LDS kernel: 16-byte chunks of 4 floats must not straddle rows or the K / N edge
    bool fast = !((((uintptr_t)A) | ((uintptr_t)B)) & 15u) && !((lda | ldb | N | K) & 3) &&
                (long long)lda * 4 * 128 + 256 < (1ll << 31) && (long long)ldb * 4 * 16 + 1024 < (1ll << 31) &&
                opt_force_config() != FORCE_GENERIC;
    const long long t128 = (long long)ceil_div(M, 128) * ceil_div(N, 128) * batch, t64 = (long long)ceil_div(M, 64) * ceil_div(N, 64) * batch;
    const long long outputs = (long long)batch * M * N;
    // 128x128 tiles once they give every other CU a block, else 64x64 (more blocks, less padding)
    bool big = t128 * 2 >= kNumCU && M >= 128 && N >= 128, elementwise = false;
    // K slices where the tiles leave more than half of the CUs idle and K is long: partial sums to the
    // library's workspace of the stream (this call has no workspace argument), summed in slice order
    int least = choose_split(big ? t128 : t64, K, 512);
    // tiles on the edge of C are stored through 31-bit offsets
    if (fast && ((M % (big ? 128 : 64)) || (N % (big ? 128 : 64))) && (least > 1 ? N : ldc) >= ge::EDGE_LDC_MAX) fast = false;
    if (!fast) {
        // rows shorter than a 16-byte chunk, or panels beyond 31-bit byte offsets: every element under its own test
        elementwise = K < 4 || N < 4 || (long long)lda * 4 * 128 + 256 >= (1ll << 31) || (long long)ldb * 4 * 32 + 1024 >= (1ll << 31) ||
                      ldc >= ge::EDGE_LDC_MAX;
        // sliced by their 128 tiles whichever tile they get: a chain of sums over all of K is less exact than its slices,
        // 8e-7 against 4e-7 at K = 2049, and no faster, 48 against 49 us
        least = choose_split(t128, K, 512);
        // Operands of any alignment: the tile whose rounds of blocks on the CUs take the matrix pipe less time (a 128 tile is
        // four of the small one, at 1.1 times its rate; 64 against 128, us: 1023 x 771 x 2049 48 / 57, 1501^3 82 / 114, 2001 x
        // 2003 x 401 45 / 42).  Fewer than 16 tiles in slices keep the large one though it is the slower, which is what they report and tests of that tile
        // count on (130 x 257 x 2075 10.3 / 15.2, 67 x 45 x 2051 7.9 / 13.5, 191 x 255 x 4097 13.1 / 20.1).  Without slices few tiles go to gemm_f32_few.h, whichever this is.
        // The others are the small tile's (255 x 255 x 1001 in slices 24 / 73, 320 x 320 x 4095 16.4 / 49.7).
        big = !elementwise && ((t64 < 16 && least > 1) ||
                               (double)((t128 + kNumCU - 1) / kNumCU) * 3.6 <= (double)((t64 + kNumCU - 1) / kNumCU));
    }
    slice_k(K, 16, least > 1 ? f32_slices(big ? 128 : 64, big ? t128 : t64, outputs, K, least, elementwise) : 1, &p.splitK, &p.kPerSlice);
    const int bm = big ? 128 : 64;
    p.tilesM = ceil_div(M, bm);
    p.tilesN = ceil_div(N, bm);
    p.groupM = choose_group_m(p.tilesM, p.tilesN);
    const long long tiles = (long long)p.tilesM * p.tilesN * batch;
    if (tiles * p.splitK > 0x7fffffffll) return GE_ERR_SHAPE;
    const bool raw = p.splitK > 1;
    void *ws = nullptr;
    int perPass = p.splitK;
    p.sliceStride = outputs;
    if (raw) {
        st = acquire_workspace(partial_bytes(M, N, batch, p.splitK), nullptr, 0, hs, &ws);
        // Room for fewer slices' partial tiles is enough, down to the least count (the library's buffer, where it cannot grow now: in a
        // capture): the slices then come as many at a time as it holds, behind the sum of those before them, with the same additions in the
        // same order, two launches a pass (us a replay: 256 x 256 x 1024, 16 slices, 9.1 at once, room for 15 14.5, 8 19.9, 4 32, the least, 2, 87;
        // 1023 x 771 x 2049, 6 slices, 46.6, 5 63.6, 4 65.8).
        int atLeast, perLeast;
        slice_k(K, 16, least, &atLeast, &perLeast);
        while (st == GE_ERR_WORKSPACE && perPass > atLeast) st = acquire_workspace(partial_bytes(M, N, batch, --perPass), nullptr, 0, hs, &ws);
        if (st != GE_OK) return st;
    }
    // few tiles and no slices: smaller ones (gemm_f32_few.h), for rows of a chunk or more and panels within 31-bit byte offsets; one step of the
    // direct-to-LDS kernel (K <= 16) is over as soon (5 x 40 x 8 3.1 us, 3.2 there)
    const int few = raw || elementwise || (fast && K <= 16) || opt_force_config() != FORCE_NONE || K < 4 || N < 4 || (long long)lda * 128 + 1024 >= (1ll << 31) || (long long)ldb * 1024 + 1024 >= (1ll << 31) ? 0
                  : ge::few_tile_f32((long long)ceil_div(M, 16) * ceil_div(N, 16) * batch, (long long)ceil_div(M, 32) * ceil_div(N, 32) * batch, K);
    const bool edge = (M % bm) || (N % bm) || (K % 16);
    auto launch_few = [&](GemmParams pg) {
        pg.tilesM = ceil_div(M, few);
        pg.tilesN = ceil_div(N, few);
        pg.groupM = choose_group_m(pg.tilesM, pg.tilesN);
        const dim3 grid((unsigned)((long long)pg.tilesM * pg.tilesN * batch)), block(256);
        const bool one = K <= ge::few_step_f32(few);
        if (few == 16) {
            if (one) GE_LAUNCH((ge::gemm_f32_few_kernel<16, 1>), grid, block, 0, hs, pg);
            else     GE_LAUNCH((ge::gemm_f32_few_kernel<16, 2>), grid, block, 0, hs, pg);
        } else {
            if (one) GE_LAUNCH((ge::gemm_f32_few_kernel<32, 1>), grid, block, 0, hs, pg);
            else     GE_LAUNCH((ge::gemm_f32_few_kernel<32, 2>), grid, block, 0, hs, pg);
        }
    };
    auto launch_tiles = [&](const GemmParams &pg) {
        const dim3 grid((unsigned)(tiles * pg.splitK)), block(256);
        auto by_edge = [&](auto bt, auto rawC) {
            constexpr int BT = decltype(bt)::value;
            constexpr bool RAW = decltype(rawC)::value;
            if (edge) GE_LAUNCH((ge::gemm_f32_fast_kernel<BT, BT, true, RAW>), grid, block, 0, hs, pg);
            else      GE_LAUNCH((ge::gemm_f32_fast_kernel<BT, BT, false, RAW>), grid, block, 0, hs, pg);
        };
        auto any_alignment = [&](auto bt, auto elements) {
            constexpr int BT = decltype(bt)::value;
            constexpr bool E = decltype(elements)::value;
            if (raw) GE_LAUNCH((ge::gemm_f32_ragged_kernel<BT, true, E>), grid, block, 0, hs, pg);
            else     GE_LAUNCH((ge::gemm_f32_ragged_kernel<BT, false, E>), grid, block, 0, hs, pg);
        };
        using Tile64 = std::integral_constant<int, 64>;
        using Tile128 = std::integral_constant<int, 128>;
        if (fast) {
            if (big) { if (raw) by_edge(Tile128{}, std::true_type{}); else by_edge(Tile128{}, std::false_type{}); }
            else     { if (raw) by_edge(Tile64{}, std::true_type{});  else by_edge(Tile64{}, std::false_type{}); }
        } else if (elementwise) {
            any_alignment(Tile64{}, std::true_type{});
        } else if (big) {
            any_alignment(Tile128{}, std::false_type{});
        } else {
            any_alignment(Tile64{}, std::false_type{});
        }
    };
    // one pass over all of K, its slices in one pass, or in several
    static const char *const names[5][3] = {{"f32_64x64x16_w4", "f32_64x64x16_w4_splitk", "f32_64x64x16_w4_splitk_passes"},
                                            {"f32_128x128x16_w4", "f32_128x128x16_w4_splitk", "f32_128x128x16_w4_splitk_passes"},
                                            {"f32_ragged_64x64x32", "f32_ragged_64x64x32_splitk", "f32_ragged_64x64x32_splitk_passes"},
                                            {"f32_ragged_128x128x32", "f32_ragged_128x128x32_splitk", "f32_ragged_128x128x32_splitk_passes"},
                                            {"f32_elements_64x64x32", "f32_elements_64x64x32_splitk", "f32_elements_64x64x32_splitk_passes"}};
    g_last_config = names[elementwise ? 4 : (fast ? 0 : 2) + (big ? 1 : 0)][!raw ? 0 : perPass == p.splitK ? 1 : 2];
    if (few) g_last_config = few == 16 ? "f32_few_16x16x256" : "f32_few_32x32x128";
    if (!raw) {
        if (few) launch_few(p);
        else     launch_tiles(p);
        return ge_host::take_launch_error() != hipSuccess ? GE_ERR_LAUNCH : GE_OK;
    }
    for (int done = 0; done < p.splitK;) {
        const int carried = done > 0 ? 1 : 0, now = std::min(perPass - carried, p.splitK - done);
        const long long skip = (long long)done * p.kPerSlice;
        GemmParams pg = p, pr = p;
        pg.A = (const float *)p.A + skip;
        pg.B = (const float *)p.B + skip * ldb;
        pg.bytesA -= 4 * skip;
        pg.bytesB -= 4 * skip * ldb;
        pg.K = (int)(K - skip);
        pg.splitK = now;
        pg.C = (float *)ws + carried * outputs;
        pg.ldc = N;
        pg.strideC = (long long)M * N;
        launch_tiles(pg);
        if (ge_host::take_launch_error() != hipSuccess) return GE_ERR_LAUNCH;
        done += now;
        pr.splitK = carried + now;
        if (done < p.splitK) {                           // the sum so far, in the first partial tile's place
            pr.C = (float *)ws;
            pr.ldc = N;
            pr.strideC = (long long)M * N;
            pr.bias = nullptr;
            pr.alpha = 1.0f;
            pr.act = GE_ACT_NONE;
        }
        if (launch_reduce(pr, ws, true, hs) != hipSuccess) return GE_ERR_LAUNCH;
    }
    return GE_OK;
}

size_t gemm_epilogue_workspace_bytes(int M, int N, int K, int batch, ge_plan_t plan, int split_k)
{
    if (M < 1 || N < 1 || K < 1 || batch < 1) return 0;
    Plan pl;
    // the tile choice (hence the slice count) depends on whether the fast
    // kernels apply; report the larger of the two answers
    size_t need = 0;
    for (int fast = 0; fast < 2; ++fast) {
        for (int other = 0; other < 2; ++other) {         // the tall-skinny kernel beside the fast ones, the ragged one beside the guarded
            if (make_plan_bf16(M, N, K, batch, fast != 0, plan, split_k, &pl, other != 0, other != 0) != GE_OK) continue;
            const size_t b = partial_bytes(M, N, batch, pl.splitK);
            if (b > need) need = b;
        }
    }
    return need;
}

int gemm_epilogue_auto_split_k(int M, int N, int K, int batch)
{
    if (M < 1 || N < 1 || K < 1 || batch < 1) return 0;
    Plan pl;
    if (make_plan_bf16(M, N, K, batch, true, GE_PLAN_AUTO, 0, &pl, true) != GE_OK) return 0;
    return pl.splitK;
}

ge_status_t ge_release_workspace(void)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return GE_ERR_WORKSPACE;
    std::lock_guard<std::mutex> lock(g_ws_mutex);
    for (std::vector<Workspace> *list : {&g_ws, &g_ws_retired}) {
        size_t kept = 0;
        for (Workspace &w : *list) {
            if (w.dev == dev) (void)hipFree(w.ptr);
            else (*list)[kept++] = w;
        }
        list->resize(kept);
    }
    return GE_OK;
}

ge_status_t ge_set_option(const char *name, const char *value)
{
    if (!name) return GE_ERR_NULL;
    if (std::strcmp(name, "force_config") == 0) {
        const int f = parse_force(value);
        if (f < 0) return GE_ERR_CONFIG;
        g_opt_force = f;
    } else if (std::strcmp(name, "waves") == 0) {
        if (value && std::strcmp(value, "8") != 0 && std::strcmp(value, "4") != 0) return GE_ERR_CONFIG;
        g_opt_waves8 = (value && std::strcmp(value, "8") == 0) ? 1 : 0;
    } else if (std::strcmp(name, "stage_k") == 0) {
        if (value && std::strcmp(value, "32") != 0 && std::strcmp(value, "64") != 0) return GE_ERR_CONFIG;
        g_opt_stage32 = (value && std::strcmp(value, "32") == 0) ? 1 : 0;
    } else if (std::strcmp(name, "conv_halo") == 0) {
        const int h = parse_halo(value);
        if (h < 0) return GE_ERR_CONFIG;
        g_opt_halo = h;
    } else {
        return GE_ERR_CONFIG;
    }
    return GE_OK;
}

const char *ge_status_string(ge_status_t status)
{
    switch (status) {
    case GE_OK: return "ok";
    case GE_ERR_NULL: return "A, B or C is NULL";
    case GE_ERR_SHAPE: return "M, N, K and batch must be >= 1 and fit the index range";
    case GE_ERR_LD: return "leading dimension smaller than the row length";
    case GE_ERR_ACT: return "unknown activation";
    case GE_ERR_ALIGN: return "pointer not aligned to its element size";
    case GE_ERR_WORKSPACE: return "split-K workspace missing, too small, misaligned or not allocatable";
    case GE_ERR_LAUNCH: return "kernel launch failed";
    case GE_ERR_CONFIG: return "unknown plan or split count";
    case GE_ERR_EPILOGUE: return "clamp bounds out of order or unknown element type";
    }
    return "unknown status";
}

const char *ge_last_config(void) { return g_last_config; }

}  // extern "C"
