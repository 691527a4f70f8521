"""Tiles that hang over M or N, with K ranges that do and do not end inside a step: the stores dropped by the resource's
bounds and by the lane offset, in every kernel that leaves fp32 straight from its accumulators.  The padding of C holds
canaries (gpu_util), and ldc is odd, so that neither rows nor columns of C are aligned to anything."""
import pytest

from paper_2604_01489_amd import binding

from gpu_util import run_case, run_fused_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,waves", [("128x128", None), ("256x256", "8"), ("256x256", None)])
@pytest.mark.parametrize("M,N,K", [(257, 8, 256), (255, 264, 256), (1, 248, 288), (129, 520, 264), (272, 136, 160)])
def test_edge_tiles_plain(oracle, M, N, K, tile, waves):
    binding.set_option("force_config", tile)
    binding.set_option("waves", waves)
    for act in ("gelu_tanh", "relu"):
        run_case(oracle, "bf16", M, N, K, alpha=0.5, act=act, ldc=N + 3, seed=M + N + K)
    run_case(oracle, "bf16", M, N, 4 * K, act="none", ldc=N + 1, seed=M, plan="splitk", split_k=2)     # partial tiles


@pytest.mark.parametrize("tile,waves", [("128x128", None), ("256x256", "8"), ("256x256", None)])
@pytest.mark.parametrize("transA,transB", [(False, False), (False, True), (True, False)])
def test_edge_tiles_fused(oracle, transA, transB, tile, waves):
    binding.set_option("force_config", tile)
    binding.set_option("waves", waves)
    for M, N, K, kw in [(136, 264, 256, dict(residual="f32", pad=(0, 0, 1, 3))), (264, 136, 288, dict(residual="bf16", pad=(0, 8, 3, 1))),
                        (8, 520, 264, dict(residual="bf16", out="bf16", pad=(8, 0, 8, 8))), (272, 248, 320, dict(residual="f32", out="bf16"))]:
        run_fused_case(oracle, M, N, K, transA=transA, transB=transB, with_row_scale=True, alpha=0.5, beta=0.5, act="gelu_tanh", seed=M + K, **kw)


@pytest.mark.parametrize("M,N,K", [(65, 68, 48), (129, 196, 36), (1100, 1996, 64), (63, 4, 16)])
def test_edge_tiles_f32(oracle, M, N, K):
    run_case(oracle, "f32", M, N, K, alpha=0.5, act="gelu_tanh", ldc=N + 1, seed=M + N)
    run_case(oracle, "f32", M, N, K, act="relu", ldc=N + 3, batch=2, seed=M)
