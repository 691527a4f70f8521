// Host-side pieces shared by the translation units of the library: plan selection, the
// library-owned split-K workspace and the last-configuration string.  Defined in
// gemm_epilogue_api.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include <tuple>
#include <utility>

#include "../../include/gemm_epilogue.h"
#include "ge_device.h"

namespace ge_host {

using ge::GemmParams;

constexpr int kNumCU = 256;          // MI355X

inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

// ---- shape -> plan -------------------------------------------------------
enum TileKind { TILE_256 = 0, TILE_128 = 1, TILE_GENERIC = 2, TILE_SKINNY = 3, TILE_RAGGED_128 = 4, TILE_RAGGED_64 = 5 };

struct Plan {
    TileKind tile;
    int bm, bn, bk;
    int tilesM, tilesN;
    bool edgeMN;     // tiles hang over M or N
    int splitK;      // >= 1
    int kPerSlice;
    bool edge;       // tiles hang over M or N, or K ends inside a K step
};

extern thread_local const char *g_last_config;

// ---- launches ------------------------------------------------------------
// A launch whose result is the launch's own: hipLaunchKernel returns it directly, so neither a
// stale error somebody else left in the runtime's per-thread slot is reported as ours, nor is it
// cleared on their behalf.  GE_LAUNCH(kernel, grid, block, ldsBytes, stream, args...) records the
// first failure of the calling thread; take_launch_error() returns and clears it.
extern thread_local hipError_t g_launch_error;

template <typename... KArgs, typename Tuple, size_t... I>
inline hipError_t launch_packed(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t st, Tuple &vals,
                                std::index_sequence<I...>)
{
    void *ptrs[] = {(void *)&std::get<I>(vals)...};
    return hipLaunchKernel((const void *)kernel, grid, block, ptrs, lds, st);
}

template <typename... KArgs, typename... Args>
inline void launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t st, Args... args)
{
    static_assert(sizeof...(KArgs) == sizeof...(Args), "one argument per kernel parameter");
    std::tuple<KArgs...> vals{static_cast<KArgs>(args)...};
    const hipError_t err = launch_packed(kernel, grid, block, lds, st, vals, std::index_sequence_for<KArgs...>{});
    if (g_launch_error == hipSuccess) g_launch_error = err;
}

inline hipError_t take_launch_error()
{
    const hipError_t err = g_launch_error;
    g_launch_error = hipSuccess;
    return err;
}

#define GE_LAUNCH(...) ::ge_host::launch(__VA_ARGS__)

// ---- switches for timing runs and tests (ge_set_option in the header) ------
enum { FORCE_NONE = 0, FORCE_256 = 1, FORCE_128 = 2, FORCE_GENERIC = 3 };
int opt_force_config();   // FORCE_*
bool opt_eight_waves();   // keep full 256 x 256 tiles on the eight-wave kernel
bool opt_stage_k32();     // no 64-k load phases in the eight-wave kernel
// the halo-staged 3 x 3 convolution kernel: by the plan's rule, never, whenever the shape allows it, or
// one of its variants whenever the shape allows that one (HALO_VARIANT0 + index)
enum { HALO_AUTO = 0, HALO_OFF = 1, HALO_ON = 2, HALO_VARIANT0 = 3 };
int opt_conv_halo();

int choose_split(long long tiles, int K, int minSlice);
void slice_k(int K, int bk, int want, int *splitK, int *kPerSlice);
// Whether the kernel for operands of any alignment (gemm_ragged.h) takes a product the direct-to-LDS kernels do not:
// rows of 8 elements or more, panels (and row blocks of C) within 31-bit byte offsets, and enough work.  plain: the plain
// operator, whose guarded kernel is the shorter one on slivers.
bool ragged_ok(int M, int N, int K, int batch, int lda, bool transA, int ldb, bool transB, int ldc, bool plain = false);
// skinny: the caller can launch the tall-skinny kernel (the plain operator only), so the plan may name it; ragged:
// likewise the kernel for operands of any alignment, where `fast` is not given
ge_status_t make_plan_bf16(int M, int N, int K, int batch, bool fast, ge_plan_t plan, int split_k, Plan *out,
                           bool skinny = false, bool ragged = false);
// The same for a result whose rows are ldc elements apart.  Tiles on the edge of C leave fp32 (the result, or the partial sums
// of a K slice, rows of N) through 31-bit offsets (edge_rows): rows of EDGE_LDC_MAX elements and more take the guarded kernel
// there (250 x 4096 x 1024 with rows 2^24 apart 57 us, 21 with a branch per masked store, which costs the others 5 to 8).
// Full tiles, bf16 output and the tall-skinny kernel are stored through 64-bit addresses and stay where they are (256 rows of
// the same: 12 us).
ge_status_t make_plan_bf16_for(int M, int N, int K, int batch, bool fast, ge_plan_t plan, int split_k, int ldc, bool f32Out, Plan *out,
                               bool skinny = false, bool ragged = false);
// Whether the call goes to workgroups in the 32 x 32 tiles of gemm_small.h, with the sums of the plan: few of them (small_layout.h), the library's own choice of
// slices, panels within 31-bit byte offsets.  The plan, and with it the workspace query, stays as it is.
bool small_ok(const Plan &pl, const GemmParams &p, ge_plan_t plan);
// Such a call needs no workspace, but asks for its slices' all the same where it can, as before there were such calls: one that is given is held to the plan's size,
// and the library's buffer of the stream grows to it, on which a smaller sliced call may count that is captured afterwards (256 x 256 x 4096 behind 512 x 512 x
// 2048).  In a capture the call goes without.
ge_status_t reserve_workspace(size_t need, void *user, size_t user_bytes, hipStream_t stream);
size_t partial_bytes(int M, int N, int batch, int splitK);
int choose_group_m(int tilesM, int tilesN);
// The four-wave kernel (gemm_bf16_w4.h) takes launches of 256 x 256 tiles whose blocks walk a K range
// long enough for its deeper pipeline to pay; four_wave_edge names the variant: 0 full tiles, 1 tiles
// hanging over M or N, 2 also K ranges that are not multiples of 128.  The option "waves" = "8" keeps the eight-wave
// kernel, for timing and for its tests.
int four_wave_edge(const Plan &pl, int K);
bool four_wave_ok(const Plan &pl, int K);
// The same for the other tiled kernels, whose blocks advance `step` k per load phase (gemm_bf16_fast.h).
int tile_edge(const Plan &pl, int K, int step);
// The buffer for `need` bytes of partial results of a call on `stream`: the caller's, if it gave one
// (checked for size and alignment), else the library's buffer for (current device, stream), grown by
// hipMalloc when a larger one is first needed -- never while the stream is capturing (GE_ERR_WORKSPACE)
// and never by freeing what an earlier call was handed (outgrown buffers are kept until
// ge_release_workspace).
ge_status_t acquire_workspace(size_t need, void *user, size_t user_bytes, hipStream_t stream, void **out);

// The second pass over p.splitK partial tiles at ws (splitk_reduce.h): p is the call's, its C the result; plain: scale, bias
// and activation only, fp32 out.
hipError_t launch_reduce(const GemmParams &p, const void *ws, bool plain, hipStream_t st);

// A symmetric A given by one triangle with few output columns (gemm_symm_api.hip): whether the kernel
// that fetches every stored element once takes the call, with which super-tile width, and the bytes
// of its partial results; run_symm launches it and the second pass (p: the call's launch parameters).
struct SymmPlan {
    bool fast;
    int st, np, terms;
    size_t bytes;
};
SymmPlan plan_symm(const ge_fused_args_t &a);
ge_status_t run_symm(const ge_fused_args_t &a, const SymmPlan &plan, GemmParams p, hipStream_t hs);

// The plain operator C = act(alpha A B + bias) (row-major operands, fp32 out): what the plain
// entry points call, and what the widened one calls when none of its extras is in use.
ge_status_t run_bf16(int M, int N, int K, const uint16_t *A, int lda, const uint16_t *B, int ldb,
                     const float *bias, float alpha, ge_act_t act, float *C, int ldc, int batch,
                     ge_plan_t plan, int split_k, void *workspace, size_t workspace_bytes, void *stream);

}  // namespace ge_host
