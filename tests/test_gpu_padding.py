"""NaN and infinity beside the payload (between the end of a row and the next, and in the triangle that is not given) leave no trace: the
kernels that read 16 bytes wherever a row starts and shift or mask off what is not theirs give the same bits as with zeros there."""
import pytest

from paper_2604_01489_amd import binding

pytestmark = pytest.mark.gpu


def _padded(rows, cols, ld, dtype, poison, seed, shift=0):
    """rows x cols of N(0, 1), ld apart, `shift` elements off the alignment; NaN and infinities in turn (or zeros) everywhere else."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    flat = torch.zeros(rows * ld + shift + 16, device="cuda", dtype=dtype)
    if poison:
        flat[0::3], flat[1::3], flat[2::3] = float("nan"), float("inf"), -float("inf")
    flat[shift:shift + rows * ld].view(rows, ld)[:, :cols] = torch.randn(rows, cols, device="cuda", generator=g).to(dtype)
    return flat[shift:]


def _same(run, kernel):
    import torch
    outs = []
    for poison in (False, True):
        outs.append(run(poison))
        assert kernel in binding.last_config(), (kernel, binding.last_config())
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("transA,transB", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("M,N,K,pad,out,kernel", [(259, 261, 257, 5, "f32", "ragged_64x64"), (2051, 2049, 9, 3, "bf16", "ragged_128x128"), (131, 67, 2051, 1, "f32", "ragged"),
                                                  (259, 261, 257, 5, "bf16", "small_32x32"), (131, 67, 701, 1, "f32", "small_32x32")])
def test_bf16_any_alignment(M, N, K, pad, out, kernel, transA, transB):
    import torch
    dt = torch.bfloat16
    rowsA, colsA, rowsB, colsB = (K, M, N, K) if transA and transB else (K, M, K, N) if transA else (M, K, N, K) if transB else (M, K, K, N)

    def run(poison):
        A, B = _padded(rowsA, colsA, colsA + pad, dt, poison, 1, 1), _padded(rowsB, colsB, colsB + pad, dt, poison, 2, 3)
        C = torch.empty(M, N, device="cuda", dtype=torch.float32 if out == "f32" else dt)
        binding.gemm_epilogue_bf16_fused(M, N, K, A, colsA + pad, B, colsB + pad, C, N, transA=transA, transB=transB, act="relu",
                                         row_scale=torch.ones(M, device="cuda"))
        return C
    _same(run, kernel)


@pytest.mark.parametrize("M,N,K,kernel", [(257, 513, 35, "f32_few_32x32"), (67, 131, 301, "f32_few_16x16"), (901, 903, 301, "f32_ragged_64x64x32"), (1921, 2046, 33, "f32_ragged_128x128x32"), (130, 257, 2075, "splitk"),
                                          (300, 3, 50, "f32_elements"), (130, 515, 3, "f32_elements")])
def test_f32_any_alignment(M, N, K, kernel):
    import torch

    def run(poison):
        A, B = _padded(M, K, K + 3, torch.float32, poison, 1, 1), _padded(K, N, N + 1, torch.float32, poison, 2, 1)
        C = torch.empty(M, N, device="cuda")
        binding.gemm_epilogue_f32(M, N, K, A, K + 3, B, N + 1, None, 0.5, "none", C, N)
        return C
    _same(run, kernel)


@pytest.mark.parametrize("M,N,K,pad", [(130, 385, 511, 3), (77, 1000, 1031, 1), (9, 65, 8193, 5), (5, 17, 9, 2), (9001, 9, 1001, 3), (40, 9, 5001, 7)])
@pytest.mark.parametrize("transB", [False, True])
def test_rowsum(M, N, K, pad, transB):
    import torch
    rows, cols = (N, K) if transB else (K, N)

    def run(poison):
        A, B = _padded(M, K, K + pad, torch.bfloat16, poison, 1, 1), _padded(rows, cols, cols + pad, torch.bfloat16, poison, 2, 3)
        params, y = torch.empty(K + 1, device="cuda"), torch.empty(M, device="cuda")
        binding.gemm_rowsum_params_bf16(N, K, B, cols + pad, transB, None, params)
        binding.gemm_rowsum_bf16(M, K, A, K + pad, params, 0.5, y)
        return torch.cat([params, y])
    _same(run, "rowsum_rows")


@pytest.mark.parametrize("M,N", [(512, 1), (776, 17), (1032, 5), (520, 31)])
@pytest.mark.parametrize("structure", ["sym_lower", "sym_upper"])
def test_symmetric(M, N, structure):
    """B with columns that are no multiple of 8 and rows padded; the triangle of A that is not given holds NaN and infinities."""
    import torch

    def run(poison):
        A = _padded(M, M, M + 8, torch.bfloat16, poison, 1)
        a = A[:M * (M + 8)].view(M, M + 8)
        bad = _padded(M, 0, M + 8, torch.bfloat16, poison, 3)[:M * (M + 8)].view(M, M + 8)
        given = torch.ones(M, M + 8, device="cuda", dtype=torch.bool)
        given = given.tril() if structure == "sym_lower" else given.triu()
        a.copy_(torch.where(given, a, bad))
        B = _padded(M, N, N + 3, torch.bfloat16, poison, 2, 1)
        C = torch.empty(M, N, device="cuda")
        binding.gemm_epilogue_bf16_fused(M, N, M, A, M + 8, B, N + 3, C, N, a_structure=structure)
        return C
    _same(run, "bf16_symm")


@pytest.mark.parametrize("cin", [8, 40, 200])
def test_conv_c8(cin):
    """Channels a multiple of 8: nothing of the memory around the input and the filters enters, where taps fall into the padding."""
    import torch

    def run(poison):
        X = _padded(1, 2 * 9 * 11 * cin, 2 * 9 * 11 * cin + 8, torch.bfloat16, poison, 1, 8)[:2 * 9 * 11 * cin].view(2, 9, 11, cin)
        W = _padded(1, 136 * 9 * cin, 136 * 9 * cin + 8, torch.bfloat16, poison, 2, 8)[:136 * 9 * cin].view(136, 3, 3, cin)
        Y = torch.empty(2, 9, 11, 136, device="cuda")
        binding.conv2d_epilogue_bf16(X, W, Y, pad=(1, 1))
        return Y
    _same(run, "_c8_")
