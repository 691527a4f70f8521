"""A few rows through weights stored N x K (csrc/gemm_few_rows.h) against the CPU oracle: row counts around its images of
16 and 32, columns around its 32-row pieces, K around its 128-k stages and shorter than its ring, every consumer."""
import numpy as np
import pytest

from paper_2604_01489_amd import binding

from gpu_util import run_fused_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 15, 16, 17, 32])
def test_few_rows(oracle, M):
    image = 16 if M <= 16 else 32
    for N, K, kw in [(1031, 512, dict(residual="bf16", out="bf16", pad=(0, 0, 3, 1), act="gelu_tanh")),       # ragged columns, odd ldc
                     (512, 1032, dict(residual="f32", beta=0.5, clamp=(-0.1, 2.0), act="relu", pad=(8, 16, 1, 5))),    # a stage of one chunk
                     (8202, 120, dict(out="bf16")),                                                             # one stage, not full
                     (264, 2184, dict(batch=3, act="gelu_tanh"))]:
        _, _, _, cfg = run_fused_case(oracle, M, N, K, transB=True, alpha=0.75, with_row_scale=True, seed=M + N, **kw)
        assert cfg == f"bf16_fused_few_rows_{image}_k128_nt"


def test_few_rows_is_repeatable_and_ignores_the_padding(oracle):
    """Bit for bit the same twice; NaN in the padding of every row of A and of the weights leaves no trace."""
    import torch
    M, N, K, ld = 5, 8300, 392, 400
    A = torch.full((M, ld), float("nan"), device="cuda", dtype=torch.bfloat16)
    W = torch.full((N, ld), float("nan"), device="cuda", dtype=torch.bfloat16)
    g = torch.Generator(device="cuda").manual_seed(3)
    A[:, :K] = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    W[:, :K] = torch.randn(N, K, device="cuda", generator=g).bfloat16()
    outs = []
    for _ in range(2):
        C = torch.empty(M, N, device="cuda")
        binding.gemm_epilogue_bf16_fused(M, N, K, A, ld, W, ld, C, N, transB=True)
        torch.cuda.synchronize()
        assert binding.last_config() == "bf16_fused_few_rows_16_k128_nt"
        outs.append(C.cpu().numpy())
    assert outs[0].tobytes() == outs[1].tobytes()
    ref = A[:, :K].double() @ W[:, :K].double().t()
    # fp32 sums of K exact products of N(0, 1) values: sqrt(K) 2^-24 of their size, sqrt(K)
    assert np.abs(outs[0] - ref.cpu().numpy()).max() < 8 * K * 2.0 ** -24


@pytest.mark.parametrize("M,N,K,slices", [(16, 8192, 2048, 4), (12, 2808, 2880, 5), (32, 1024, 3072, 6), (16, 8192, 8192, 4), (5, 6144, 16384, 8),
                                          (32, 8192, 16384, 16)])
def test_few_rows_are_as_exact_as_k_slices(M, N, K, slices):
    """fp32 output: no further from the 64-bit result than the tiles with as many K slices as their plan takes or more.
    The errors are those of 32768 to 262144 outputs: their norm is steady to a percent."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    W = torch.randn(N, K, device="cuda", generator=g).bfloat16()
    ref = A.double() @ W.double().t().contiguous()
    err = {}
    for plan, kw in [("auto", {}), ("splitk", dict(split_k=slices))]:
        C = torch.empty(M, N, device="cuda")
        binding.gemm_epilogue_bf16_fused(M, N, K, A, K, W, K, C, N, transB=True, plan=plan, **kw)
        torch.cuda.synchronize()
        assert ("few_rows" in binding.last_config()) == (plan == "auto"), binding.last_config()
        err[plan] = float((C.double() - ref).norm() / ref.norm())
    assert err["auto"] <= 1.01 * err["splitk"], err


@pytest.mark.parametrize("structure", ["lower", "upper"])
@pytest.mark.parametrize("M,N,K,out", [(16, 1024, 512, "f32"), (32, 8200, 1160, "f32"), (5, 520, 2056, "bf16"), (17, 6152, 200, "f32")])
def test_few_rows_of_a_triangular_a(oracle, M, N, K, out, structure):
    """With the promise, the bits of the same call without it: the same kernel, which leaves out stages of zeros."""
    kw = dict(transB=True, alpha=0.5, act="relu", with_row_scale=True, out=out, seed=M + K, a_structure=structure)
    got, _, _, cfg = run_fused_case(oracle, M, N, K, **kw)
    plain, _, _, cfg2 = run_fused_case(oracle, M, N, K, hint=False, **kw)
    assert cfg == cfg2 and "few_rows" in cfg
    assert np.array_equal(got, plain)
