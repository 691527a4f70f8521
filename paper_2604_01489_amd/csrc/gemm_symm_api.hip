// Host side of the symmetric-operand kernel (gemm_symm.h): plan (super-tile width, workspace) and
// launches.  Called by gemm_epilogue_bf16_fused for a_structure = GE_A_SYM_LOWER / GE_A_SYM_UPPER; a
// translation unit of its own because the kernel's instantiations take minutes to compile.
#include <hip/hip_runtime.h>

#include <cstdio>

#include "../../include/gemm_epilogue.h"
#include "gemm_fused.h"
#include "gemm_symm.h"
#include "ge_host.h"

namespace ge_host {

namespace {
thread_local char g_symm_config[64];
}

// ---- symmetric A given by one triangle, few output columns: every stored element fetched once -------
SymmPlan plan_symm(const ge_fused_args_t &a)
{
    SymmPlan sp{};
    sp.fast = a.N <= 32 && a.M >= 512 && (a.M % 8) == 0 && (a.lda % 8) == 0 && !(((uintptr_t)a.A) & 15u) &&
              (long long)a.lda * 2 * ge_symm::SUB + 4096 < (1ll << 31) && opt_force_config() != FORCE_GENERIC;
    if (!sp.fast) return sp;
    sp.np = a.N <= 16 ? 16 : 32;
    // The side of the super-tiles: wider ones write fewer partial results (8 N / ST bytes per byte of A) but
    // make fewer workgroups, and what counts is the number of rounds those take on the CUs times the
    // sub-tiles of one.  Estimated cost in sub-tile loads per CU, partial results included; ties go to the
    // wider tile.  (768 with 32 columns does not fit the LDS.)
    double best = 0.0;
    for (int st : {768, 512, 256}) {
        if (st == 768 && sp.np == 32) continue;
        const long long t = ceil_div(a.M, st), blocks = t * (t + 1) / 2 * a.batch;
        const long long rounds = (blocks + kNumCU - 1) / kNumCU;
        const double ns = st / 128.0;
        const double cost = (double)rounds * ns * ns * (1.0 + 8.0 * a.N / st);
        if (best == 0.0 || cost < best) { best = cost; sp.st = st; }
    }
    sp.terms = ceil_div(a.M, sp.st);
    sp.bytes = (size_t)sp.terms * (size_t)a.batch * (size_t)a.M * (size_t)a.N * sizeof(float);
    const long long blocks = (long long)sp.terms * (sp.terms + 1) / 2;
    if (blocks > 0x7fffffffll || a.batch > 65535) sp.fast = false;
    return sp;
}

namespace {
template <int ST, int NP>
void launch_symm(const ge::SymmParams &sp, bool upper, bool bVec, dim3 grid, hipStream_t st)
{
    auto launch = [&](auto vecC, auto imageC) {
        constexpr bool BVEC = decltype(vecC)::value, IMAGE = decltype(imageC)::value;
        if (upper) GE_LAUNCH((ge::gemm_symm_bf16_kernel<ST, NP, true, BVEC, IMAGE>), grid, dim3(256), 0, st, sp);
        else       GE_LAUNCH((ge::gemm_symm_bf16_kernel<ST, NP, false, BVEC, IMAGE>), grid, dim3(256), 0, st, sp);
    };
    if (bVec) return launch(std::true_type{}, std::false_type{});
    if constexpr (NP == 32) {
        if (ge::symm_image(sp.N)) return launch(std::false_type{}, std::true_type{});
    }
    launch(std::false_type{}, std::false_type{});
}

template <int ST>
void launch_symm(const ge::SymmParams &sp, int np, bool upper, bool bVec, dim3 grid, hipStream_t st)
{
    if (np == 16) launch_symm<ST, 16>(sp, upper, bVec, grid, st);
    else          launch_symm<ST, 32>(sp, upper, bVec, grid, st);
}

}  // namespace

// p: the launch parameters of the call as the second pass needs them (epilogue, C, sizes)
ge_status_t run_symm(const ge_fused_args_t &a, const SymmPlan &plan, GemmParams p, hipStream_t hs)
{
    void *ws = nullptr;
    ge_status_t st = acquire_workspace(plan.bytes, a.workspace, a.workspace_bytes, hs, &ws);
    if (st != GE_OK) return st;
    ge::SymmParams sp{};
    sp.A = a.A; sp.B = a.B; sp.W = (float *)ws;
    sp.M = a.M; sp.N = a.N; sp.lda = a.lda; sp.ldb = a.ldb;
    sp.transB = a.transB ? 1 : 0;
    sp.upper = a.a_structure == GE_A_SYM_UPPER ? 1 : 0;
    sp.batch = a.batch;
    sp.tiles = plan.terms;
    // (the offsets of a super-tile's rows of B are 32-bit)
    const bool bVec = !a.transB && a.ldb < (1 << 20) && (a.N % 8) == 0 && (a.ldb % 8) == 0 && !(((uintptr_t)a.B) & 15u);
    sp.bytesA = 2 * (((long long)a.M - 1) * a.lda + a.M);
    // Wide super-tiles: past the 256 MB memory-side cache what it does not hold.  us, through / past, one triangle again and again and two
    // in turn: 16384 x 16, 268 MB, 57.3 / 61.3 and 69.2 / 61.6; 18432 x 16, 340 MB, 90.6 / 86.4 and 93.0 / 87.0; 15360 x 16, 236 MB,
    // 56.7 / 60.3 and 64.7 / 60.5; 11264 x 16, 127 MB, 31.7 / 35.1 and 33.1 / 36.2; 8192 x 32, 67 MB, 35.4 / 38.4.  Rows that are no whole
    // lines go through it at any size: two sub-tiles share the line between them (16848 x 16, 284 MB, 63.3 / 71.4 and 68.6 / 71.4).
    const bool lines = a.lda % 64 == 0 && !(((uintptr_t)a.A) & 127u);
    sp.past = lines && (double)a.batch * a.M * (a.M + 1.0) > 256.0 * 1024 * 1024 ? 1 : 0;
    const dim3 grid((unsigned)((long long)plan.terms * (plan.terms + 1) / 2), (unsigned)a.batch);
    const bool upper = sp.upper != 0;
    if (plan.st == 768)      launch_symm<768, 16>(sp, upper, bVec, grid, hs);
    else if (plan.st == 512) launch_symm<512>(sp, plan.np, upper, bVec, grid, hs);
    else                     launch_symm<256>(sp, plan.np, upper, bVec, grid, hs);
    if (ge_host::take_launch_error() != hipSuccess) return GE_ERR_LAUNCH;
    // the terms are the slices of the second pass: added in their order, then the consumer chain
    p.splitK = plan.terms;
    p.sliceStride = (long long)a.batch * a.M * a.N;
    if (launch_reduce(p, ws, false, hs) != hipSuccess) return GE_ERR_LAUNCH;
    std::snprintf(g_symm_config, sizeof g_symm_config, "bf16_symm_%s_%dx%d_n%d", upper ? "upper" : "lower", plan.st, plan.st, plan.np);
    g_last_config = g_symm_config;
    return GE_OK;
}

}  // namespace ge_host
