"""Convolutions whose channels are a multiple of 8 but not of 32, on the gathering kernel with a tap per 16-byte chunk, against
the CPU oracle: every number of taps a K step of 32 can span, K ranges that end inside a step, padding, strides and
dilations, both tiles, K slices, every consumer."""
import pytest

from paper_2604_01489_amd import binding

from test_gpu_conv import run_conv_case

pytestmark = pytest.mark.gpu

C8 = "conv_bf16_c8_128x128x32_w4"


@pytest.mark.parametrize("cin", [8, 16, 24, 40, 48, 56, 72, 80, 104, 200])
def test_conv_c8_channels(oracle, cin):
    cfg = run_conv_case(oracle, (2, 15, 17, cin, 136, 3, 3), pad=(1, 1), act="relu", residual="bf16", out="bf16", seed=cin)
    assert cfg.startswith(C8)          # with K slices where K is long
    cfg = run_conv_case(oracle, (9, 14, 13, cin, 72, 5, 4), stride=(1, 2), pad=(2, 0), dil=(2, 1), alpha=0.5, act="gelu_tanh", seed=cin + 1)
    assert cfg.startswith(C8)          # with K slices where K is long
    cfg = run_conv_case(oracle, (8, 21, 19, cin, 168, 1, 1), stride=(1, 1), residual="f32", beta=-0.5, clamp=(-0.5, 0.5), seed=cin + 2)
    assert cfg.startswith(C8)          # with K slices where K is long


def test_conv_c8_large_tile_and_slices(oracle):
    for waves_out in ("f32", "bf16"):
        binding.set_option("force_config", "256x256")
        cfg = run_conv_case(oracle, (2, 20, 17, 48, 264, 3, 3), pad=(1, 1), act="relu", out=waves_out, seed=5)
        assert cfg == "conv_bf16_c8_256x256x32_w8"
        binding.set_option("force_config", None)
    cfg = run_conv_case(oracle, (1, 9, 9, 200, 104, 3, 3), pad=(1, 1), act="relu", residual="bf16", out="bf16", seed=6)
    assert cfg.startswith("conv_bf16_c8_128x128x32_w4")
    cfg = run_conv_case(oracle, (1, 7, 7, 456, 128, 3, 3), pad=(1, 1), act="gelu_tanh", alpha=0.5, seed=7)
    assert cfg == "conv_bf16_c8_128x128x32_w4_splitk"
