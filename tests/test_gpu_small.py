"""Products of few output tiles in tiles of 32 x 32 (csrc/gemm_small.h).  The names of the configurations are the plan's and do not tell: which sizes take
the kernel is asserted by the host model (small_layout_check.cpp), and a test switch that keeps the plan's own kernel gives the other side."""
import os
import subprocess

import numpy as np
import pytest

from paper_2604_01489_amd import binding

from gpu_util import run_case, run_fused_case

LAYOUTS = [(False, False), (False, True), (True, False), (True, True)]


def test_small_layout_model(tmp_path):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = str(tmp_path / "small_layout_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-o", exe, os.path.join(root, "tests", "small_layout_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    assert "small layout ok" in res.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("M,N,K,kw", [
    (8, 8, 8, dict()),                                                       # a corner of one tile
    (40, 264, 256, dict(residual="bf16", batch=2)),                          # one step, edges in both directions
    (264, 232, 264, dict(residual="f32", beta=0.5, clamp=(-0.5, 1.0))),      # a second step of 8
    (72, 1096, 520, dict(residual="bf16", pad=(8, 16, 8, 8))),               # three steps
    (64, 96, 1024, dict()),                                                  # four full ones
    (136, 40, 1288, dict(residual="f32", pad=(0, 0, 3, 0))),                 # the walk's loop, a residual at any address
    (320, 768, 256, dict())])                                                # 240 tiles, full
def test_aligned(oracle, transA, transB, M, N, K, kw):
    """Same bits as the tile that the plan names: the sums are in the same order."""
    for out in ("f32", "bf16"):
        outs = []
        for option in (None, "128x128"):
            binding.set_option("force_config", option)
            got, _, _, _ = run_fused_case(oracle, M, N, K, transA=transA, transB=transB, alpha=0.75, with_row_scale=True, act="gelu_tanh", out=out,
                                          plan="direct", seed=M + K, **kw)
            outs.append(got)
        assert np.array_equal(outs[0], outs[1])
        binding.set_option("force_config", None)


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("M,N,K,kw", [(131, 261, 65, dict()), (257, 259, 257, dict(misalign=1)), (33, 517, 263, dict(pad=(1, 3, 2, 5), residual="bf16")),
                                      (193, 129, 513, dict(misalign=3, batch=2, residual="f32")), (100, 333, 900, dict(pad=(0, 0, 1, 1)))])
def test_any_alignment(oracle, transA, transB, M, N, K, kw):
    for out in ("f32", "bf16"):
        run_fused_case(oracle, M, N, K, transA=transA, transB=transB, alpha=0.5, with_row_scale=True, act="relu", out=out, plan="direct", seed=M + N, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,kw", [(44, 690, 1109, dict()), (131, 67, 1792, dict(misalign=1)), (512, 512, 2048, dict()), (144, 440, 2560, dict())])
def test_in_place_of_k_slices(oracle, M, N, K, kw):
    """In runs of steps no longer than the plan's slices: as exact as these, and nothing goes to a workspace, so a capture needs none."""
    import torch
    run_case(oracle, "bf16", M, N, K, alpha=K ** -0.5, act="gelu_tanh", seed=M + K, plan="auto", **kw)
    g = torch.Generator(device="cuda").manual_seed(K)
    A, B = torch.randn(M, K, device="cuda", generator=g).bfloat16(), torch.randn(K, N, device="cuda", generator=g).bfloat16()
    ref = A.double() @ B.double()
    err, C = {}, torch.empty(M, N, device="cuda")
    for plan in ("auto", "splitk"):
        binding.gemm_epilogue_bf16_ex(M, N, K, A, K, B, N, None, 1.0, "none", C, N, plan=plan)
        torch.cuda.synchronize()
        err[plan] = float((C.double() - ref).norm() / ref.norm())
    # 30000 outputs and more: the norm of the errors is steady to two percent
    assert err["auto"] <= 1.02 * err["splitk"], err
    eager, side = torch.empty(M, N, device="cuda"), torch.cuda.Stream()
    binding.gemm_epilogue_bf16(M, N, K, A, K, B, N, None, 1.0, "none", eager, N)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        binding.gemm_epilogue_bf16(M, N, K, A, K, B, N, None, 1.0, "none", C, N, stream=side)
    for _ in range(3):
        C.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, eager)


@pytest.mark.gpu
def test_a_workspace_that_was_too_small_still_is():
    import torch
    M, N, K = 512, 512, 2048
    A, B, C = (torch.zeros(n, device="cuda", dtype=t) for n, t in ((M * K, torch.bfloat16), (K * N, torch.bfloat16), (M * N, torch.float32)))
    need = binding.workspace_bytes(M, N, K)
    with pytest.raises(binding.GemmEpilogueError):
        binding.gemm_epilogue_bf16_ex(M, N, K, A, K, B, N, None, 1.0, "none", C, N, workspace=torch.empty(1024, device="cuda"))
    binding.gemm_epilogue_bf16_ex(M, N, K, A, K, B, N, None, 1.0, "none", C, N, workspace=torch.empty(need // 4, device="cuda"))
    torch.cuda.synchronize()
