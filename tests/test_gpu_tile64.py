"""The 64 x 128 tile for few blocks and the one-phase kernels for K <= 64 (csrc/gemm_tile64_launch.h): the bits of the 128 x 128 tile, which a test switch keeps.  Which calls take which is
asserted by the host model (small_layout_check.cpp), that these do by the configuration's name."""
import numpy as np
import pytest

from paper_2604_01489_amd import binding

from gpu_util import run_case, run_fused_case, takes_small
from test_gpu_conv import run_conv_case

pytestmark = pytest.mark.gpu

LAYOUTS = [(False, False), (False, True), (True, False), (True, True)]


def _both(run, kernel):
    """The same bits from ``kernel`` (None: the call takes none of these) as from the switch's tile."""
    outs = [run()]
    binding.set_option("force_config", "128x128")
    outs.append(run())
    binding.set_option("force_config", None)
    assert kernel in outs[0][3] if kernel else not takes_small(outs[0][3]), outs[0][3]
    assert "128x128x" in outs[1][3], outs[1][3]
    assert np.array_equal(outs[0][0], outs[1][0])


def _blocks(M, N, batch=1):
    return -(-M // 64) * -(-N // 128) * batch


def _short(M, N, out, batch=1):
    """The one-phase kernel of a product whose plan names the 128 x 128 tile."""
    blocks = _blocks(M, N, batch)
    if out == "bf16":
        return "128x128_k64" if 768 < blocks <= 1024 or blocks > 4096 else "64x128_k64"
    return "64x128_k64" if blocks <= 256 or 1024 < blocks <= (4096 if -(-M // 64) % 2 else 1280) else None


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("M,N,K,kw", [
    (1024, 2048, 320, dict()),                                                       # 256 full tiles
    (584, 1288, 264, dict(residual="bf16", beta=0.5)),                               # edges in both directions, K ends inside a step
    (72, 5000, 520, dict(residual="f32", pad=(8, 16, 3, 8), clamp=(-0.5, 1.0))),     # one tile row and a little
    (520, 1032, 1280, dict(batch=2)),                                                # a ring that goes round ten times
    (1500, 2000, 104, dict(residual="bf16")), (1024, 2048, 128, dict(batch=5))])      # more than a block a CU (bf16 out)
def test_ring(oracle, transA, transB, M, N, K, kw):
    for out in ("f32", "bf16"):
        ring = (out == "bf16" or _blocks(M, N, kw.get("batch", 1)) <= 256) and not (transA and M % 8)
        _both(lambda: run_fused_case(oracle, M, N, K, transA=transA, transB=transB, alpha=0.75, with_row_scale=True, act="gelu_tanh", out=out, plan="direct", seed=M + K, **kw),
              "64x128x32_w4" if ring else None)


@pytest.mark.parametrize("transA,transB", LAYOUTS)
@pytest.mark.parametrize("M,N,K,batch,kw", [
    (128, 256, 64, 40, dict()),                                      # full tiles, both steps
    (200, 136, 40, 33, dict(residual="bf16")),                       # the second step ends in a chunk
    (72, 264, 32, 60, dict(residual="f32", pad=(8, 8, 1, 8))),       # one step
    (264, 136, 8, 50, dict()),                                       # one chunk
    (256, 512, 64, 260, dict(residual="bf16"))])                     # more than sixteen 64 x 128 tiles to a CU: the wide one
def test_short_k(oracle, transA, transB, M, N, K, batch, kw):
    for out in ("bf16", "f32"):
        _both(lambda: run_fused_case(oracle, M, N, K, batch=batch, transA=transA, transB=transB, alpha=0.5, with_row_scale=True, act="relu", out=out, plan="direct", seed=M + K, **kw),
              _short(M, N, out, batch))


@pytest.mark.parametrize("M,N,K,batch", [(1000, 1928, 296, 1), (512, 512, 48, 30), (136, 264, 64, 300)])
@pytest.mark.parametrize("act", ["none", "relu", "gelu_tanh"])
def test_plain_operator(oracle, M, N, K, batch, act):
    _both(lambda: run_case(oracle, "bf16", M, N, K, batch=batch, alpha=0.5, act=act, seed=M + K), _short(M, N, "f32", batch) if K <= 64 else "64x128x32_w4")


RING, SHORT, WIDE = "64x128x32_w4", "64x128_k64_w4", "128x128_k64_w4"


@pytest.mark.parametrize("shape,kw,f32,bf16", [
    ((12, 24, 24, 96, 128, 3, 3), dict(pad=(1, 1), residual="bf16", beta=0.5), RING, RING),             # 108 row tiles, 27 steps
    ((3, 41, 39, 32, 200, 3, 3), dict(pad=(1, 1), stride=(2, 1), residual="f32"), RING, RING),          # edges in both directions
    ((9, 30, 31, 40, 136, 3, 3), dict(pad=(1, 1), residual="bf16"), None, RING),                        # channels a multiple of 8: K ends inside a step
    ((6, 32, 32, 72, 512, 3, 1), dict(pad=(1, 0), dil=(2, 1)), None, RING),                             # ... more than a block a CU
    ((5, 56, 56, 128, 256, 1, 1), dict(act="gelu_tanh"), None, RING),                                   # four steps, two blocks a CU
    ((6, 28, 28, 32, 136, 1, 1), dict(residual=None), SHORT, SHORT),                                    # one step in one phase, less than a block a CU
    ((20, 28, 28, 64, 136, 1, 1), dict(residual="f32"), None, SHORT),                                   # two
    ((40, 28, 28, 64, 136, 1, 1), dict(residual="bf16"), None, WIDE),                                   # on the wide tile, four a CU
    ((40, 28, 29, 24, 136, 1, 1), dict(), None, WIDE),                                                  # ... K = 24
    ((45, 56, 56, 32, 256, 1, 1), dict(act="relu"), None, WIDE)])                                       # ... more than sixteen
def test_convolution(oracle, shape, kw, f32, bf16):
    for out, kernel in (("f32", f32), ("bf16", bf16)):
        run = lambda: run_conv_case(oracle, shape, out=out, seed=sum(shape), **{"act": "relu", **kw})
        prefix = "conv_bf16_c8_" if shape[3] % 32 else "conv_bf16_"
        cfg = run()
        assert cfg == prefix + kernel if kernel else not takes_small(cfg), cfg
        binding.set_option("force_config", "128x128")
        cfg = run()
        binding.set_option("force_config", None)
        assert cfg == prefix + "128x128x32_w4", cfg
