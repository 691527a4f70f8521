"""The 64 x 128 tile for few blocks and the one-phase kernels for K <= 64 (csrc/gemm_tile64_launch.h): the bits of the plan's own tile, which a test switch keeps.  The names of the
configurations are the plan's: which calls take which is asserted by the host model (small_layout_check.cpp)."""
import numpy as np
import pytest

from paper_2604_01489_amd import binding

from gpu_util import run_case, run_fused_case
from test_gpu_conv import run_conv_case

pytestmark = pytest.mark.gpu

LAYOUTS = [(False, False), (False, True), (True, False), (True, True)]


def _both(run):
    outs = [run()]
    binding.set_option("force_config", "256x256" if "256x256" in outs[0][3] else "128x128")
    outs.append(run())
    binding.set_option("force_config", None)
    assert outs[0][3] == outs[1][3], (outs[0][3], outs[1][3])
    assert np.array_equal(outs[0][0], outs[1][0])


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("M,N,K,kw", [
    (1024, 2048, 320, dict()),                                                       # 256 full tiles
    (584, 1288, 264, dict(residual="bf16", beta=0.5)),                               # edges in both directions, K ends inside a step
    (72, 5000, 520, dict(residual="f32", pad=(8, 16, 3, 8), clamp=(-0.5, 1.0))),     # one tile row and a little
    (520, 1032, 1280, dict(batch=2)),                                                # a ring that goes round ten times
    (1500, 2000, 104, dict(residual="bf16")), (1024, 2048, 128, dict(batch=5))])      # more than a block a CU (bf16 out)
def test_ring(oracle, transA, transB, M, N, K, kw):
    for out in ("f32", "bf16"):
        _both(lambda: run_fused_case(oracle, M, N, K, transA=transA, transB=transB, alpha=0.75, with_row_scale=True, act="gelu_tanh", out=out, plan="direct", seed=M + K, **kw))


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("M,N,K,batch,kw", [
    (128, 256, 64, 40, dict()),                                      # full tiles, both steps
    (200, 136, 40, 33, dict(residual="bf16")),                       # the second step ends in a chunk
    (72, 264, 32, 60, dict(residual="f32", pad=(8, 8, 1, 8))),       # one step
    (264, 136, 8, 50, dict()),                                       # one chunk
    (256, 512, 64, 260, dict(residual="bf16"))])                     # more than sixteen 64 x 128 tiles to a CU: the wide one
def test_short_k(oracle, transA, transB, M, N, K, batch, kw):
    for out in ("bf16", "f32"):
        run_fused_case(oracle, M, N, K, batch=batch, transA=transA, transB=transB, alpha=0.5, with_row_scale=True, act="relu", out=out, plan="direct", seed=M + K, **kw)


@pytest.mark.parametrize("M,N,K,batch", [(1000, 1928, 296, 1), (512, 512, 48, 30), (136, 264, 64, 300)])
@pytest.mark.parametrize("act", ["none", "relu", "gelu_tanh"])
def test_plain_operator(oracle, M, N, K, batch, act):
    _both(lambda: run_case(oracle, "bf16", M, N, K, batch=batch, alpha=0.5, act=act, seed=M + K))


@pytest.mark.parametrize("shape,kw", [
    ((8, 24, 24, 96, 128, 3, 3), dict(pad=(1, 1), residual="bf16", beta=0.5)),             # 72 row tiles, 27 steps
    ((3, 41, 39, 32, 200, 3, 3), dict(pad=(1, 1), stride=(2, 1), residual="f32")),         # edges in both directions
    ((9, 30, 31, 40, 136, 3, 3), dict(pad=(1, 1), residual="bf16")),                       # channels a multiple of 8: K ends inside a step
    ((6, 32, 32, 72, 512, 3, 1), dict(pad=(1, 0), dil=(2, 1))),                            # ... more than a block a CU
    ((5, 56, 56, 128, 256, 1, 1), dict(act="gelu_tanh")),                                  # four steps, two blocks a CU
    ((40, 28, 28, 64, 136, 1, 1), dict(residual="bf16")),                                  # K = 64 in one phase
    ((40, 28, 29, 24, 136, 1, 1), dict()),                                                 # ... K = 24
    ((45, 56, 56, 32, 256, 1, 1), dict(act="relu"))])                                      # ... the wide one
def test_convolution(oracle, shape, kw):
    for out in ("f32", "bf16"):
        assert run_conv_case(oracle, shape, out=out, seed=sum(shape), **{"act": "relu", **kw}) in ("conv_bf16_128x128x32_w4", "conv_bf16_c8_128x128x32_w4", "conv_bf16_256x256x32_w8")
