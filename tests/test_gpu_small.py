"""Products of few output tiles in tiles of 32 x 32 (csrc/gemm_small.h).  Which sizes take the kernel is asserted by the host model (small_layout_check.cpp), that these do by the
configuration's name, and a test switch that keeps the plan's own kernel gives the other side."""
import os
import subprocess

import numpy as np
import pytest

from paper_2604_01489_amd import binding

from gpu_util import run_case, run_fused_case
from test_gpu_conv import run_conv_case

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
            got, _, _, cfg = run_fused_case(oracle, M, N, K, transA=transA, transB=transB, alpha=0.75, with_row_scale=True, act="gelu_tanh", out=out,
                                            plan="direct", seed=M + K, **kw)
            outs.append(got)
            assert ("small_32x32" if option is None else "128x128") in cfg, cfg
        assert np.array_equal(outs[0], outs[1])
        binding.set_option("force_config", None)


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("M,N,K,kw", [(131, 261, 65, dict()), (257, 259, 257, dict(misalign=1)), (33, 517, 263, dict(pad=(1, 3, 2, 5), residual="bf16")),
                                      (193, 129, 513, dict(misalign=3, batch=2, residual="f32")), (100, 333, 900, dict(pad=(0, 0, 1, 1)))])
def test_any_alignment(oracle, transA, transB, M, N, K, kw):
    for out in ("f32", "bf16"):
        outs = []
        oddA, oddB = [(mis + ld) % 2 == 1 or mis % 2 == 1 for mis, ld in ((kw.get("misalign", 0), (M if transA else K) + kw.get("pad", (0, 0))[0]),
                                                                            (kw.get("misalign", 0), (K if transB else N) + kw.get("pad", (0, 0))[1]))]
        odd = oddA and (oddB or "residual" not in kw) if transA else oddA and oddB and "residual" not in kw
        stays = out == "f32" and odd and 256 < K <= 320                            # on the 64 x 64 tile
        for option in (None, "128x128"):
            binding.set_option("force_config", option)
            got, _, _, cfg = run_fused_case(oracle, M, N, K, transA=transA, transB=transB, alpha=0.5, with_row_scale=True, act="relu", out=out, plan="direct", seed=M + N, **kw)
            outs.append(got)
            assert ("small_32x32" if option is None and not stays else "ragged_64x64") in cfg, cfg
        binding.set_option("force_config", None)
        assert np.array_equal(outs[0], outs[1])


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,kw", [(44, 690, 1109, dict()), (131, 67, 1536, dict(misalign=1)), (512, 512, 2048, dict()), (144, 440, 2560, dict())])
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
        assert binding.last_config() == "bf16_small_32x32x256" if plan == "auto" else binding.last_config().endswith("_splitk"), binding.last_config()
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


@pytest.mark.gpu
def test_a_sliced_call_captured_behind_one_that_slices_no_longer():
    """The first call adds up its slices in its workgroups, and the stream's buffer grows to them all the same: the capture of a call that parks less finds room."""
    import torch
    g, side = torch.Generator(device="cuda").manual_seed(3), torch.cuda.Stream()

    def operands(M, N, K):
        return [torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((M, K), (K, N))] + [torch.empty(M, N, device="cuda") for _ in range(2)]
    for conv in (False, True):
        assert binding.load().ge_release_workspace() == 0                      # no buffer left of an earlier test
        A, B, C, _ = operands(512, 512, 2048)
        if conv:
            X, W = torch.randn(4, 14, 14, 256, device="cuda", generator=g).bfloat16(), torch.randn(256, 3, 3, 256, device="cuda", generator=g).bfloat16()
            Y = torch.empty(4, 14, 14, 256, device="cuda")
        A2, B2, C2, eager = operands(256, 256, 4096)
        binding.gemm_epilogue_bf16(256, 256, 4096, A2, 4096, B2, 256, None, 1.0, "none", eager, 256)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            if conv: binding.conv2d_epilogue_bf16(X, W, Y, pad=(1, 1))
            else: binding.gemm_epilogue_bf16(512, 512, 2048, A, 2048, B, 512, None, 1.0, "none", C, 512)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            binding.gemm_epilogue_bf16(256, 256, 4096, A2, 4096, B2, 256, None, 1.0, "none", C2, 256, stream=side)
        for _ in range(3):
            C2.fill_(-1.0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(C2, eager)
        del graph


@pytest.mark.gpu
@pytest.mark.parametrize("shape,kw", [
    ((4, 17, 15, 8, 40, 3, 3), dict(pad=(1, 1))),                                                  # a tap to a chunk
    ((2, 15, 17, 24, 136, 3, 3), dict(pad=(1, 1), residual="bf16", out="bf16")),                    # one step of 216, taps that end inside a chunk's neighbours
    ((9, 14, 13, 40, 72, 5, 4), dict(stride=(1, 2), pad=(2, 0), dil=(2, 1), act="gelu_tanh")),      # four steps, every way the geometry enters
    ((2, 20, 20, 64, 64, 3, 3), dict(pad=(1, 1), out="bf16")),                                      # 576: three steps
    ((3, 9, 9, 256, 40, 1, 1), dict(residual="f32", beta=-0.5, clamp=(-0.5, 0.5))),                 # one full step, no padding
    ((4, 9, 9, 128, 96, 3, 3), dict(pad=(0, 2), stride=(3, 2), out="bf16")),                        # 1152: five
    ((1, 12, 12, 256, 128, 3, 3), dict(pad=(1, 1), residual="bf16", out="bf16")),                   # 2304, in place of slices
    ((1, 11, 9, 264, 96, 3, 3), dict(pad=(1, 1)))])                                                 # 2376 of channels a multiple of 8
def test_convolutions(oracle, shape, kw):
    outs = []
    for option in (None, "128x128"):
        binding.set_option("force_config", option)
        kw2 = dict(kw)
        outs.append(run_conv_case(oracle, shape, alpha=0.75, act=kw2.pop("act", "relu"), seed=sum(shape), **kw2))
    assert "small_32x32" in outs[0] and "128x128" in outs[1], outs


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,cin,cout", [(1, 14, 256, 96), (2, 9, 264, 128)])
def test_convolutions_are_as_exact_as_slices(n, h, cin, cout):
    """3 x 3, K of 2304 and 2376 in place of slices (the switch keeps the plan's tile and its slices).  18000 outputs and more: the norm of the errors is
    steady to two percent."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(cin)
    X, W = torch.randn(n, h, h, cin, device="cuda", generator=g).bfloat16(), torch.randn(cout, 3, 3, cin, device="cuda", generator=g).bfloat16()
    x = torch.nn.functional.pad(X.double(), (0, 0, 1, 1, 1, 1))
    ref = sum(x[:, i:i + h, j:j + h, :].reshape(-1, cin) @ W[:, i, j, :].double().t().contiguous() for i in range(3) for j in range(3))
    err = {}
    for option in (None, "128x128"):
        binding.set_option("force_config", option)
        Y = torch.empty(n, h, h, cout, device="cuda")
        binding.conv2d_epilogue_bf16(X, W, Y, pad=(1, 1))
        torch.cuda.synchronize()
        assert "small_32x32" in binding.last_config() if option is None else binding.last_config().endswith("_splitk"), binding.last_config()
        err[option] = float((Y.reshape(-1, cout).double() - ref).norm() / ref.norm())
    assert err[None] <= 1.02 * err["128x128"], err
