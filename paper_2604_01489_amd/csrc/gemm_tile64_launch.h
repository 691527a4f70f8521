// Two more tiles of gemm_bf16_kernel (gemm_bf16_fast.h) for calls whose plan names the 128 x 128 or the 256 x 256 one and takes no K slices: 64 x 128 where that
// gives every block a CU of its own, and K <= 64 in one load phase and half the LDS, so that three and more blocks share a CU.  Same sums in the same order.
//
// 64 x 128: the 128 x 128 tile on fewer than 128 CUs spends 8.3 us beside its steps (0.17 to 0.21 us each), this one 5.0 and 0.15 to 0.17, as its epilogue is half as
// long, and there are twice as many of them: B K x N, bf16 out, 1024 x 1536 x 1216 14.8 -> 10.6 us; of 870 drawn calls each 0.74 to 0.92 of the time.  More
// blocks than CUs: three of them are on a CU at once, where two of the larger tile are, and what that saves is the epilogue.  K <= 128, bf16 out, of 1300 drawn calls up to three to a CU
// 0.88 to 0.92, a fourth 1.12, up to six 0.85 to 0.89; beside the 256 x 256 tile five 0.91; fp32 out 0.92 to 0.96 with single ones 1.05; K = 192 0.98, 1024 1.1 (1280 x 2560 x
// 1024, 400 blocks, 13.6 / 15.0).
// Convolutions: a block a CU 0.69 to 0.82 of the time (8 images of 56 x 56 x 128 -> 128, 3 x 3, stride 2, 15.3 -> 11.5 us); beyond, K <= 128 as above 0.80 to 0.91; channels a multiple of 8 only, up
// to two blocks a CU K = 576 0.87, up to one and a half 1152 0.85 (490 blocks of K = 720 17.6 / 18.6), up to six K = 256 0.83 to 0.92 (else K = 256 0.95, 576 1.0); K <= 64 0.71 to 0.97.
// K <= 64, bf16 out: 256 of 256 x 256 x 64 13.8 -> 11.5 us, 256 of 128 x 128 x 64 6.0 -> 5.4, 256 of 512 x 512 x 64, there on 128 x 128 tiles in place of 256 x 256 ones (64 x 128: 46.6), 49.6 -> 43.6, as
// a fourth to a CU is (209 of 80 x 256 x 40 6.55 us, 64 x 128 6.80; convolutions 0.97);
// with fp32 out, where the stores are all, 0.93 of the time up to a block a CU, between one and four none (0.96 to 0.99), the fifth 0.84 to 0.91.  Beyond that where half of the larger
// tile's last row of blocks is padding (64-row tiles odd in number), up to sixteen: 0.81 to 0.94, results that come from memory 0.87 to 0.97 (1500 drawn calls each).  Rows of whole larger tiles
// only gain while the 256 MB cache holds what is written (0.88 to 0.97 up to ten a CU); from memory 0.96 to 1.03, with a residual 0.97 to 1.08, one call in three by more than 3 %.
// bf16 out beyond sixteen to a CU, 128 x 128 against 64 x 128, 470 drawn calls: up to 6000 blocks 1.05, with a residual 1.08 to 1.09; up to 10000 1.00, 1.06; 256 of 512 x 512 x 64, 8192
// blocks, 43.6 / 46.6: the line is drawn for full tiles, the others (either way faster than the ring of four stages, 0.79 to 0.94) would gain on the narrower one.
#pragma once
#include <hip/hip_runtime.h>

#include "ge_device.h"
#include "ge_host.h"
#include "small_layout.h"

namespace ge_host {

// Which of them a call takes (small_layout.h), whatever tile its plan names.
using ge::Tile64;
using ge::TILE64_NO;
using ge::TILE64_RING;
using ge::TILE64_SHORT_WIDE;
Tile64 tile64_of(const Plan &pl, const ge::GemmParams &p, ge_plan_t plan);
enum { TILE64_PLAIN = 0, TILE64_CONV = 1, TILE64_CONV_C8 = 2 };
const char *tile64_config(Tile64 kind, int family);     // its configuration's name

// For the storages of p.transA / p.transB and the output type of p.cType; p.tilesM, p.tilesN and p.groupM are set here.
void launch_tile64(ge::GemmParams p, Tile64 kind, hipStream_t st);
void launch_tile64_conv(ge::GemmParams p, Tile64 kind, bool c8, hipStream_t st);     // p.transA 0, p.transB 1
dim3 tile64_grid(ge::GemmParams &p, bool wide);
void launch_tile64_ring(const ge::GemmParams &p, dim3 grid, hipStream_t st);
void launch_tile64_short(const ge::GemmParams &p, bool wide, dim3 grid, hipStream_t st);

}  // namespace ge_host
