"""The bf16 kernel for operands of any alignment (csrc/gemm_ragged.h) against the CPU oracles, on sizes around its tiles
(64 and 128) and its 64-k steps, with rows that start at any 2-byte address, in every operand storage, output type and
slicing of K.  Products of up to 2^20 multiply-adds stay on the guarded kernel.  The padding
of the operands holds huge finite values and the last row ends where the allocation's payload ends (gpu_util)."""
import os
import subprocess

import pytest

from paper_2604_01489_amd import binding

from gpu_util import both_kernels, run_case, run_fused_case, takes_small

LAYOUTS = [(False, False), (False, True), (True, False), (True, True)]
NAME = {(False, False): "nn", (False, True): "nt", (True, False): "tn", (True, True): "tt"}


def test_ragged_layout_model(tmp_path):
    """Host model of the loads and the LDS image, from the kernel's own index header."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = str(tmp_path / "ragged_layout_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-o", exe, os.path.join(root, "tests", "ragged_layout_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    assert "ragged layout ok" in res.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,tile,small", [
    (257, 259, 257, "64x64", False),         # one over the tiles and the steps
    (321, 383, 191, "64x64", True),          # full tiles but for the last, one short of three steps
    (9, 4099, 513, "64x64", True),           # a sliver of one tile row
    (4099, 9, 513, "64x64", True),           # B's rows barely a chunk long
    (901, 1021, 513, "64x64", False),        # more tiles than the kernel for few takes, one k over the steps
    (2049, 2047, 9, "128x128", False),       # one step, a chunk and one element
    (2175, 2050, 67, "128x128", False),      # one element over two tiles and a step
])
def test_ragged_plain(oracle, M, N, K, tile, small):
    both_kernels(lambda: run_case(oracle, "bf16", M, N, K, alpha=0.5, act="gelu_tanh", seed=M + N + K)[3].replace("_splitk", ""), f"bf16_ragged_{tile}x64", small)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,batch,tile", [(9, 4099, 41, 16, "64x64"), (48, 2316, 33, 16, "64x64"), (2316, 48, 33, 16, "64x64"),
                                              (129, 129, 33, 60, "64x64"), (67, 131, 41, 200, "128x128")])
def test_ragged_tile_of_slivers(oracle, M, N, K, batch, tile):
    """Many tiles of which most is padding: the small ones, where a large one takes the place of fewer than two and a half."""
    _, _, _, cfg = run_case(oracle, "bf16", M, N, K, batch=batch, alpha=0.5, act="relu", seed=M + N, misalign=1)
    assert cfg == f"bf16_ragged_{tile}x64"


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", LAYOUTS)
def test_ragged_layouts(oracle, transA, transB):
    for M, N, K, kw in [(300, 301, 259, dict(pad=(1, 3, 2, 5), residual="f32", beta=0.5, clamp=(-0.1, 2.0), act="gelu_tanh")),
                        (263, 519, 129, dict(out="bf16", residual="bf16", beta=-0.5, act="relu", pad=(0, 0, 1, 3), misalign=1)),
                        (256, 512, 128, dict(out="bf16", residual="f32", misalign=3, pad=(0, 8, 1, 0))),
                        (136, 137, 301, dict(batch=3, out="bf16", act="gelu_tanh", misalign=1)),
                        # more tiles than the kernel for few takes: several steps, a residual and odd rows in every storage
                        (601, 605, 301, dict(out="bf16", residual="bf16", beta=-0.5, misalign=1)),
                        (600, 607, 257, dict(residual="f32", pad=(1, 3, 2, 5), act="gelu_tanh"))]:
        both_kernels(lambda: run_fused_case(oracle, M, N, K, transA=transA, transB=transB, alpha=0.75, with_row_scale=True, plan="direct", seed=M + N, **kw)[3],
                     f"bf16_fused_ragged_64x64x64_{NAME[transA, transB]}", small=M < 600)
    for M, N, K, out in [(2063, 2049, 65, "bf16"), (2048, 2051, 70, "f32")]:
        _, _, _, cfg = run_fused_case(oracle, M, N, K, transA=transA, transB=transB, with_row_scale=True, act="relu", out=out, plan="direct",
                                      seed=M + K)
        assert cfg == f"bf16_fused_ragged_128x128x64_{NAME[transA, transB]}"


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", LAYOUTS)
def test_ragged_k_slices(oracle, transA, transB):
    """Slices that end inside a step, in slice order, bit for bit the same twice."""
    outs = []
    for _ in range(2):
        got, _, _, cfg = run_fused_case(oracle, 131, 67, 2051, transA=transA, transB=transB, alpha=1.0 / 32, with_row_scale=True,
                                        act="relu", out="bf16", plan="splitk", split_k=3, seed=7)
        assert cfg == f"bf16_fused_ragged_64x64x64_{NAME[transA, transB]}_splitk"
        outs.append(got.tobytes())
    assert outs[0] == outs[1]


@pytest.mark.gpu
@pytest.mark.parametrize("structure", ["lower", "upper"])
def test_ragged_triangular(oracle, structure):
    """Blocks whose K range ends at, or starts inside, their own tile; some of them empty."""
    for M, N, K in [(331, 197, 331), (131, 401, 517), (517, 401, 131)]:
        for transA in (False, True):
            kw = dict(transA=transA, transB=True, alpha=0.5, act="relu", seed=M, a_structure=structure, plan="direct")
            got, _, _, cfg = run_fused_case(oracle, M, N, K, **kw)
            assert "ragged" in cfg
            plain, _, _, cfg = run_fused_case(oracle, M, N, K, hint=False, **kw)       # the bits of the call without the promise
            assert ("ragged" in cfg or takes_small(cfg)) and (got == plain).all()
            if takes_small(cfg):                                                       # and on the tile that the promise keeps
                binding.set_option("force_config", "128x128")
                plain, _, _, cfg = run_fused_case(oracle, M, N, K, hint=False, **kw)
                binding.set_option("force_config", None)
                assert "ragged" in cfg and (got == plain).all()


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,cfg", [
    (257, 513, 33, "f32_ragged_64x64x32"),            # one over the tiles and a 32-k step
    (323, 517, 31, "f32_ragged_64x64x32"),            # one step, not full
    (321, 518, 95, "f32_ragged_64x64x32"),            # three steps
    (1000, 130, 5, "f32_ragged_64x64x32"),            # barely more than a chunk of k
    (901, 903, 301, "f32_ragged_64x64x32"),           # more tiles than the kernel for few takes
    (2047, 1922, 33, "f32_ragged_128x128x32"),
    (1921, 2046, 66, "f32_ragged_128x128x32"),
    (300, 3, 50, "f32_elements_64x64x32"),              # rows of B shorter than a chunk
    (130, 515, 3, "f32_elements_64x64x32"),             # rows of A shorter than a chunk
    (70, 3, 1100, "f32_elements_64x64x32_splitk"),
    (257, 515, 1061, "f32_ragged_64x64x32_splitk"),   # slices that end inside a step
])
def test_f32_any_alignment(oracle, M, N, K, cfg):
    """fp32 operands of any alignment (csrc/gemm_f32_ragged.h): odd sizes, odd leading dimensions, pointers off by 4 bytes."""
    for kw in [dict(), dict(misalign=1, lda=K + 1, ldb=N + 3, ldc=N + 2)]:
        both_kernels(lambda: run_case(oracle, "f32", M, N, K, alpha=0.5, act="gelu_tanh", seed=M + N + K, **kw)[3], cfg, small=M * N < 200000 and "elements" not in cfg and "splitk" not in cfg)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,out", [(520, 776, 384, "f32"), (264, 1032, 456, "bf16"), (136, 2056, 1160, "bf16"), (72, 1096, 1160, "bf16")])
def test_small_tiles_of_aligned_operands(oracle, M, N, K, out):
    """Few tiles and K of 384 or more: the 64 x 64 tiles, with the same sums as the larger ones in the same order."""
    outs = []
    for option in (None, "128x128"):
        binding.set_option("force_config", option)
        got, _, _, cfg = run_fused_case(oracle, M, N, K, transB=True, act="gelu_tanh", residual="bf16", out=out, plan="auto" if option is None else "direct", seed=M)
        outs.append(got)
        assert ("small_32x32" if M == 72 else "ragged_64x64x64") in cfg if option is None else "128x128" in cfg, cfg
    assert (outs[0] == outs[1]).all()
    # a promised triangular A stays on the larger tiles, with the bits of the call without the promise on these
    kw = dict(transB=True, with_row_scale=True, out=out, seed=N)
    binding.set_option("force_config", None)
    for structure in ("lower", "upper"):
        got, _, _, cfg = run_fused_case(oracle, M, N, K, a_structure=structure, **kw)
        plain, _, _, cfg2 = run_fused_case(oracle, M, N, K, a_structure=structure, hint=False, **kw)
        assert "ragged" not in cfg and ("small_32x32" if M == 72 else "ragged_64x64x64") in cfg2 and (got == plain).all(), (cfg, cfg2)
