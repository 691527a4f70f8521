"""Convolutions whose channels are a multiple of 8 but not of 32, on the gathering kernel with a tap per 16-byte chunk, against
the CPU oracle: every number of taps a K step of 32 can span, K ranges that end inside a step, padding, strides and
dilations, both tiles, K slices, every consumer."""
import pytest

from paper_2604_01489_amd import binding

from gpu_util import both_kernels
from test_gpu_conv import run_conv_case

pytestmark = pytest.mark.gpu

C8 = "conv_bf16_c8_128x128x32_w4"


@pytest.mark.parametrize("cin", [8, 16, 24, 40, 48, 56, 72, 80, 104, 200])
def test_conv_c8_channels(oracle, cin):
    # (with K slices where K is long: more than 2560 stays in slices)
    both_kernels(lambda: run_conv_case(oracle, (2, 15, 17, cin, 136, 3, 3), pad=(1, 1), act="relu", residual="bf16", out="bf16", seed=cin).replace("_splitk", ""), C8)
    both_kernels(lambda: run_conv_case(oracle, (9, 14, 13, cin, 72, 5, 4), stride=(1, 2), pad=(2, 0), dil=(2, 1), alpha=0.5, act="gelu_tanh",
                                       seed=cin + 1).replace("_splitk", ""), C8, small=cin * 20 <= 2560)
    both_kernels(lambda: run_conv_case(oracle, (8, 21, 19, cin, 168, 1, 1), stride=(1, 1), residual="f32", beta=-0.5, clamp=(-0.5, 0.5), seed=cin + 2), C8)


def test_conv_c8_large_tile_and_slices(oracle):
    for waves_out in ("f32", "bf16"):
        binding.set_option("force_config", "256x256")
        cfg = run_conv_case(oracle, (2, 20, 17, 48, 264, 3, 3), pad=(1, 1), act="relu", out=waves_out, seed=5)
        assert cfg == "conv_bf16_c8_256x256x32_w8"
        binding.set_option("force_config", None)
    both_kernels(lambda: run_conv_case(oracle, (1, 9, 9, 200, 104, 3, 3), pad=(1, 1), act="relu", residual="bf16", out="bf16", seed=6).replace("_splitk", ""), C8)
    cfg = run_conv_case(oracle, (1, 7, 7, 456, 128, 3, 3), pad=(1, 1), act="gelu_tanh", alpha=0.5, seed=7)
    assert cfg == "conv_bf16_c8_128x128x32_w4_splitk"


@pytest.mark.parametrize("shape", [(1, 9, 9, 200, 104, 3), (1, 14, 14, 120, 64, 3), (2, 14, 14, 80, 128, 5), (4, 7, 7, 1160, 256, 1)])
def test_conv_c8_is_as_exact_as_the_guarded_kernel(shape):
    """fp32 output where the guarded kernel slices K: no further from the 64-bit result (errors of 8424 and more outputs, whose norm is
    steady to two percent)."""
    import torch
    n, h, w, cin, cout, k = shape
    g = torch.Generator(device="cuda").manual_seed(cin)
    X = torch.randn(n, h, w, cin, device="cuda", generator=g).bfloat16()
    W = torch.randn(cout, k, k, cin, device="cuda", generator=g).bfloat16()
    x = torch.nn.functional.pad(X.double(), (0, 0) + (k // 2,) * 4)
    ref = torch.zeros(n * h * w, cout, device="cuda", dtype=torch.float64)
    for i in range(k):
        for j in range(k):
            ref += x[:, i:i + h, j:j + w, :].reshape(n * h * w, cin) @ W[:, i, j, :].double().t().contiguous()
    err = {}
    for option in (None, "generic"):
        binding.set_option("force_config", option)
        Y = torch.empty(n, h, w, cout, device="cuda")
        binding.conv2d_epilogue_bf16(X, W, Y, pad=(k // 2, k // 2))
        torch.cuda.synchronize()
        assert ("_c8_" in binding.last_config()) == (option is None), binding.last_config()
        err[option] = float((Y.reshape(-1, cout).double() - ref).norm() / ref.norm())
    assert err[None] <= 1.02 * err["generic"], err
