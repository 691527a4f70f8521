"""Row sum: the blocks of the row pass around the widths of their sweeps and the number of rows that fills the CUs, and the column
pass around the rows that it has on their way."""
import numpy as np
import pytest

from paper_2604_01489_amd import binding, inputs as gen

pytestmark = pytest.mark.gpu


def _run(M, N, K, transB, lda=None, ldb=None):
    import torch
    lda, ldb = lda or K, ldb or (K if transB else N)
    A = gen.to_bf16_bits(gen.normal(M + K, gen.STREAM_A, M * K, K ** -0.5).reshape(M, K))
    B = gen.to_bf16_bits(gen.normal(N + K, gen.STREAM_B, N * K, 1.0).reshape((N, K) if transB else (K, N)))
    bias = gen.uniform(N, gen.STREAM_BIAS, N, -0.1, 0.1)

    def padded(x, ld):                                   # NaN beyond the rows' payload
        full = np.full((x.shape[0], ld), 0x7FC0, np.uint16)
        full[:, :x.shape[1]] = x
        return torch.from_numpy(full.view(np.int16)).to("cuda:0")

    dA, dB, dbias = padded(A, lda), padded(B, ldb), torch.from_numpy(bias).to("cuda:0")
    params = torch.full((K + 1,), float("nan"), device="cuda:0")
    y = torch.full((M,), float("nan"), device="cuda:0")
    binding.gemm_rowsum_params_bf16(N, K, dB, ldb, transB, dbias, params)
    binding.gemm_rowsum_bf16(M, K, dA, lda, params, 0.5, y)
    torch.cuda.synchronize()
    f64 = lambda bits: (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    s = np.append(f64(B).sum(0 if transB else 1), bias.astype(np.float64).sum())
    # fp32 sums of fp32 terms, in chains of at most 64 under trees: a few parts in 10^7 of the norm
    assert np.linalg.norm(params.cpu().numpy() - s) <= 1e-6 * np.linalg.norm(s)
    ref = 0.5 * (f64(A) @ s[:-1]) + s[-1]
    assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-6 * np.linalg.norm(ref)
    return binding.last_config()


@pytest.mark.parametrize("M,K", [(1, 384), (33, 512), (31, 520), (17, 1024), (15, 1032), (9, 2048), (7, 2056), (4095, 2056), (4096, 2056), (4097, 2048),
                                 (8, 4096), (1, 8200), (4103, 4104),
                                 # nearly one block of 16 waves to a CU, and one row beyond or short of that
                                 (2048, 2568), (2049, 2568), (2304, 2560), (2305, 2560), (4096, 2064), (6144, 1032), (6145, 1032), (8192, 2048), (8193, 2048)])
def test_rows_around_a_sweep(M, K):
    assert _run(M, 40, K, True) == "rowsum_rows_wide"
    if K >= 2048 and M < 1000:
        assert _run(M, 40, K + 1, True) == "rowsum_rows_wide_any"
    if K > 2051 and M > 4000:
        assert _run(M, 24, K - 3, True, lda=K + 5) == "rowsum_rows_wide_any"


@pytest.mark.parametrize("N", [1, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33, 40, 47, 48, 63, 64, 65, 79, 127])
def test_columns_by_number_of_rows(N):
    for K in (384, 391):
        _run(16, N, K, True)
    _run(24, N, 2056, True, ldb=2064)


def test_long_chunks():
    """Chunks of 64, 32 and 16 rows, the last one of any length."""
    for N, K in [(8192 + 5, 8192), (4096 + 33, 4099), (2048 + 11, 2048), (777, 1024)]:
        _run(64, N, K, True)


def test_row_of_nearly_2_31_columns():
    """The kernel of one wave a row at the end of its longest aligned row: the columns behind the last whole piece, and none in front of
    the row."""
    import torch
    N, ld = 2 ** 31 - 9, 2 ** 31 - 8
    B = torch.zeros(ld + 128, dtype=torch.bfloat16, device="cuda:0")
    B[:128] = float("nan")                                # in front of the row
    row = B[128:]
    row[N - 80:N] = 1.0
    row[N:] = float("nan")
    row[0] = 2.0
    params = torch.full((2,), float("nan"), device="cuda:0")
    binding.gemm_rowsum_params_bf16(N, 1, row, ld, False, None, params)
    torch.cuda.synchronize()
    assert binding.last_config() == "rowsum_params_rows"
    assert params.tolist() == [82.0, 0.0]
