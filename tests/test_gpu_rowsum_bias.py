"""The bias sum that the first block of a row pass takes on (weights stored K x N): every kernel of the pass, lengths around one load of 256 threads and around eight of them."""
import pytest

from paper_2604_01489_amd import binding

from test_gpu_rowsum import run_rowsum_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,N,kw", [
    (37, 1, dict()), (9, 255, dict()), (700, 257, dict(misalign=1)),                 # one wave a row: short, aligned or not
    (2100, 384, dict()), (1030, 2047, dict(misalign=1)), (300, 2056, dict()),        # four waves; any alignment; eight waves
    (4000, 2304, dict()), (2300, 4096, dict()), (5, 6145, dict(with_bias=False))])   # blocks of 16 waves; no bias
def test_bias_sum(oracle, K, N, kw):
    _, cfg, _ = run_rowsum_case(oracle, 33, N, K, transB=False, alpha=0.5, seed=K + N, **kw)
    assert cfg == "rowsum_params_rows"


def test_one_launch(oracle):
    """Captured, the call is one kernel: replays give what the eager call gives."""
    import torch
    B = torch.randn(640, 1024, device="cuda:0").to(torch.bfloat16).view(torch.int16)
    bias = torch.randn(1024, device="cuda:0")
    want, got = torch.zeros(641, device="cuda:0"), torch.zeros(641, device="cuda:0")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        binding.gemm_rowsum_params_bf16(1024, 640, B, 1024, False, bias, want)
        side.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            binding.gemm_rowsum_params_bf16(1024, 640, B, 1024, False, bias, got)
        for _ in range(3):
            got.zero_()
            g.replay()
            side.synchronize()
            assert torch.equal(got, want)
