"""K slices of fp32 products: as many as fill the CUs, never fewer than before; and a buffer that holds fewer partial tiles
than the call would write (the library's, inside a capture, where it cannot grow) gives the same bits."""
import numpy as np
import pytest

from paper_2604_01489_amd import binding, inputs as gen

pytestmark = pytest.mark.gpu


def _operands(M, N, K, batch, seed):
    import torch
    A = gen.uniform(seed, gen.STREAM_A, batch * M * K, -1, 1).reshape(batch, M, K)
    B = gen.uniform(seed, gen.STREAM_B, batch * K * N, -1, 1).reshape(batch, K, N)
    bias = gen.uniform(seed, gen.STREAM_BIAS, N, -1, 1)
    return A, B, bias, [torch.from_numpy(x).to("cuda:0") for x in (A, B, bias)]


@pytest.mark.parametrize("M,N,K,batch,kernel", [
    (255, 257, 1025, 1, "f32_ragged_64x64x32_splitk"),        # 25 tiles, the shortest K that is sliced
    (67, 45, 2051, 1, "f32_ragged_128x128x32_splitk"),        # one tile of 128, slices of 64 and a few k
    (129, 300, 1031, 3, "f32_ragged_64x64x32_splitk"),        # batches
    (256, 192, 1024, 1, "f32_64x64x16_w4_splitk"),            # aligned, full tiles
    (200, 136, 2076, 1, "f32_64x64x16_w4_splitk"),            # aligned, tiles on the edge, K ends inside a step
    (300, 3, 1500, 1, "f32_elements_64x64x32_splitk"),
])
def test_slices_against_64_bits(M, N, K, batch, kernel):
    import torch
    A, B, bias, (dA, dB, dbias) = _operands(M, N, K, batch, M + N + K)
    C = torch.empty(batch, M, N, device="cuda:0")
    for _ in range(2):
        C.fill_(float("nan"))
        binding.gemm_epilogue_f32(M, N, K, dA, K, dB, N, dbias, 0.5, "relu", C, N, batch)
        torch.cuda.synchronize()
        assert binding.last_config() == kernel, binding.last_config()
        ref = np.maximum(0.5 * np.matmul(A.astype(np.float64), B.astype(np.float64)) + bias, 0.0)
        # sums of 1024 and more terms in chains of at most 512: well below 1e-6 of the norm
        assert np.linalg.norm(C.cpu().numpy() - ref) <= 1e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("M,N,K,aligned", [(1023, 771, 2049, False), (320, 320, 4096, True)])
def test_same_bits_from_a_buffer_with_room_for_fewer_slices(M, N, K, aligned):
    """The capture stream's buffer is made by another call (4 or 8 slices of bf16 operands): too small for this one's partial tiles."""
    import torch
    A, B, bias, (dA, dB, dbias) = _operands(M, N, K, 1, 5)
    eager, out = torch.empty(M, N, device="cuda:0"), torch.empty(M, N, device="cuda:0")
    binding.gemm_epilogue_f32(M, N, K, dA, K, dB, N, dbias, 0.5, "gelu_tanh", eager, N)
    torch.cuda.synchronize()
    least = 4 if not aligned else 8
    side = torch.cuda.Stream()
    H = torch.zeros(1024, 4096, dtype=torch.bfloat16, device="cuda:0")
    C2 = torch.empty(M, 1024, device="cuda:0")
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        # least slices of M x N, rounded up to the 8 columns that aligned bf16 operands want
        cols = (N + 7) // 8 * 8
        binding.gemm_epilogue_bf16_ex(M, cols, 4096, H, 4096, H, 1024, None, 1.0, "none", C2, 1024, plan="splitk", split_k=least, stream=side)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            binding.gemm_epilogue_f32(M, N, K, dA, K, dB, N, dbias, 0.5, "gelu_tanh", out, N, stream=side)
    torch.cuda.synchronize()
    for _ in range(3):
        out.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)


@pytest.mark.parametrize("M,N,K,room", [
    (256, 256, 1024, 2),            # two slices, then one at a time behind the carried sum
    (256, 256, 1024, 5),            # five, then four at a time, then what is left
    (256, 256, 1024, 15),           # all but one
    (255, 255, 20000, 38),         # 39 slices asked for at least, 38 after rounding
    (67, 45, 2051, 4),
])
def test_slices_a_few_at_a_time(M, N, K, room):
    """A capture on a stream whose buffer has room for `room` partial tiles and no more: taken down to the least count, in as many passes
    as that makes, with the bits of the eager call."""
    import torch
    binding.release_workspace()           # (pooled streams come with buffers of earlier tests)
    A, B, bias, (dA, dB, dbias) = _operands(M, N, K, 1, 5)
    eager, out = torch.empty(M, N, device="cuda:0"), torch.empty(M, N, device="cuda:0")
    binding.gemm_epilogue_f32(M, N, K, dA, K, dB, N, dbias, 0.5, "gelu_tanh", eager, N)
    torch.cuda.synchronize()
    whole = binding.last_config()
    side = torch.cuda.Stream()
    H = torch.zeros(256, 64 * room, dtype=torch.bfloat16, device="cuda:0")
    W = torch.zeros(64 * room, 256, dtype=torch.bfloat16, device="cuda:0")
    C2 = torch.empty(M, N, device="cuda:0")
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        binding.gemm_epilogue_bf16_ex(M, N, 64 * room, H, 64 * room, W, 256, None, 1.0, "none", C2, N, plan="splitk", split_k=room, stream=side)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            binding.gemm_epilogue_f32(M, N, K, dA, K, dB, N, dbias, 0.5, "gelu_tanh", out, N, stream=side)
            captured = binding.last_config()
    assert whole.endswith("_splitk") and captured == whole + "_passes", (whole, captured)
    torch.cuda.synchronize()
    for _ in range(3):
        out.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
