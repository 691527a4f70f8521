"""fp32 products of few tiles in tiles of 16 x 16 or 32 x 32 (csrc/gemm_f32_few.h).  Which sizes take which tile is asserted by the host model (small_layout_check.cpp), that these
take it by the configuration's name."""
import pytest

from paper_2604_01489_amd import binding

from gpu_util import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,kw", [
    (4, 4, 4, dict()),                                  # a corner of one tile, one chunk
    (64, 96, 64, dict()),                               # 32: one step, half of it
    (33, 517, 61, dict(batch=2)),                       # 32: edges, a step that ends in a chunk
    (48, 272, 72, dict()),                              # 16: one step of which the last two waves have little or nothing
    (17, 35, 255, dict(batch=7)),                       # 16: one short of a step
    (256, 256, 256, dict()),                            # 16: one full step, a tile to every CU
    (80, 100, 512, dict()),                             # 16: two steps
    (131, 257, 515, dict(misalign=1)),                  # 16: three, rows at any address
    (142, 343, 983, dict(lda=985, ldb=347, ldc=345)),   # 16: four
    (250, 444, 1020, dict()),                           # 16, four full but for a chunk
    (300, 700, 129, dict(misalign=3)),                  # 32: two steps, the second of one k
    (256, 938, 347, dict()),                            # 32: three
    (500, 510, 640, dict()),                            # 32: five full ones
    (480, 1056, 1023, dict(misalign=1))])               # 32: eight, two tiles to a CU
@pytest.mark.parametrize("act", ["none", "gelu_tanh"])
def test_few_tiles(oracle, M, N, K, kw, act):
    t16 = -(-M // 16) * -(-N // 16) * kw.get("batch", 1)
    kernel = "f32_64x64x16_w4" if K <= 16 else "f32_few_16x16x256" if K > 64 and t16 <= (512 if K > 128 else 256) else "f32_few_32x32x128"
    outs = [run_case(oracle, "f32", M, N, K, alpha=0.5, act=act, seed=M + N + K, **kw) for _ in range(2)]
    assert outs[0][0].tobytes() == outs[1][0].tobytes() and outs[0][3] == kernel, outs[0][3]


@pytest.mark.parametrize("M,N,K", [(256, 256, 256), (256, 250, 1000), (512, 512, 512), (500, 500, 1000), (255, 938, 347), (512, 500, 60)])
def test_as_exact_as_the_larger_tiles(M, N, K):
    """Against 64 bits, beside the one chain over K of the 64 x 64 tiles (the switch that keeps aligned operands from their kernel keeps these from the small tiles
    as well): four chains of a quarter each have about half the error where it is many steps long.  64000 outputs and more: the norm of the errors is steady to a percent."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(K)
    A, B = torch.rand(M, K, device="cuda", generator=g) * 2 - 1, torch.rand(K, N, device="cuda", generator=g) * 2 - 1
    ref = A.double() @ B.double()
    err = {}
    for option in (None, "generic"):
        binding.set_option("force_config", option)
        C = torch.empty(M, N, device="cuda")
        binding.gemm_epilogue_f32(M, N, K, A, K, B, N, None, 1.0, "none", C, N)
        torch.cuda.synchronize()
        err[option] = float((C.double() - ref).norm() / ref.norm())
    binding.set_option("force_config", None)
    assert err[None] <= (0.6 if K >= 256 else 1.01) * err["generic"], err
