"""Wide super-tiles of the symmetric kernel (512 and 768) on batches of matrices that are no multiple of them: every way the blocks of B
are brought in (16-byte pieces straight into LDS, any address through registers, stored N x K) and the terms leave (whole fours of
columns, the one to three behind them, through their image in LDS), both triangles, the other one filled with NaN.  Reference: the mirrored matrices in fp64."""
import pytest

from paper_2604_01489_amd import binding

pytestmark = pytest.mark.gpu

# width -> batch, M that the plan gives it (csrc/gemm_symm_api.hip); the last super-tile hangs over
SIZES = {512: (24, 1800), 768: (12, 4360)}


@pytest.fixture(scope="module")
def stored():
    """The arrays by width and triangle: the stored one N(0, 1 / M), the other one NaN."""
    import torch
    made = {}

    def get(width, uplo):
        if (width, uplo) not in made:
            made.clear()
            torch.cuda.empty_cache()
            batch, M = SIZES[width]
            g = torch.Generator(device="cuda").manual_seed(width)
            A = torch.randn(batch, M, M, generator=g, device="cuda").mul_(M ** -0.5).to(torch.bfloat16)
            keep = torch.ones(M, M, device="cuda", dtype=torch.bool)
            keep = keep.tril() if uplo == "lower" else keep.triu()
            made[width, uplo] = A.masked_fill_(~keep, float("nan"))
        return made[width, uplo]
    return get


@pytest.mark.parametrize("uplo", ["lower", "upper"])
@pytest.mark.parametrize("width,columns", [(512, (1, 3, 5, 10, 15, 16, 24, 31, 32)), (768, (1, 2, 5, 7, 8, 12, 14))])
def test_wide_super_tiles(stored, width, columns, uplo):
    import torch
    batch, M = SIZES[width]
    A = stored(width, uplo)
    for N in columns:
        g = torch.Generator(device="cuda").manual_seed(N)
        B = torch.randn(batch, M, N, generator=g, device="cuda").to(torch.bfloat16)
        ref = []
        for a, b in zip(A, B):
            t = torch.nan_to_num(a.double())
            t = t.tril() if uplo == "lower" else t.triu()
            ref.append((t + t.t() - torch.diag(t.diagonal())).contiguous() @ b.double())
        ref = torch.stack(ref)
        for transB, pad, shift in [(False, 0, 0), (False, 3, 0), (False, 8 - N % 8, 1), (True, 0, 0), (True, 5, 1)]:
            rows = B.transpose(1, 2).contiguous() if transB else B
            ldb = rows.shape[2] + pad
            held = torch.full((rows.numel() // rows.shape[2] * ldb + shift,), float("nan"), device="cuda", dtype=torch.bfloat16)
            dB = held[shift:]
            dB.view(batch, rows.shape[1], ldb)[:, :, :rows.shape[2]] = rows
            C = torch.full((batch, M, N), float("nan"), device="cuda")
            print(f"symmetric {width} {uplo} M={M} N={N} batch={batch} transB={transB} ldb={ldb} shift={shift}", flush=True)
            binding.gemm_epilogue_bf16_fused(M, N, M, A, M, dB, ldb, C, N, batch=batch, transB=transB, a_structure="sym_" + uplo)
            torch.cuda.synchronize()
            assert binding.last_config() == f"bf16_symm_{uplo}_{width}x{width}_n{16 if N <= 16 else 32}", binding.last_config()
            # fp32 sums of M exact products in chains of at most a super-tile's width: a few parts in 10^7 of the norm
            assert float((C.double() - ref).norm()) <= 1e-6 * float(ref.norm())
