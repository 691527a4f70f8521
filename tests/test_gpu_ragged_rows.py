"""bf16 operands whose rows start at odd elements: each row is put together from 4-byte addresses (csrc/gemm_ragged.h).  Rows all
odd, every other one odd, one operand only; and the small products of more than 2^20 multiply-adds, which take the same kernel.  The names do not
tell four waves from eight: which calls take which is asserted by the host model (ragged_rows_check.cpp)."""
import os
import subprocess

import pytest

from paper_2604_01489_amd import binding

from gpu_util import both_kernels, run_case, run_fused_case


def test_ragged_rows_model(tmp_path):
    """Host model of the reads and the LDS image, from the kernel's own index header."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = str(tmp_path / "ragged_rows_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-o", exe, os.path.join(root, "tests", "ragged_rows_check.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    assert "ragged rows ok" in res.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", [(False, False), (False, True), (True, False), (True, True)])
def test_rows_at_odd_elements(oracle, transA, transB):
    tile = {True: "128x128", False: "64x64"}
    for M, N, K, large, kw in [
            (200, 136, 328, False, dict(misalign=1, pad=(0, 0, 0, 0))),        # every row odd
            (200, 136, 328, False, dict(pad=(1, 0, 0, 0))),                    # A alone, every other row
            (200, 136, 328, False, dict(pad=(0, 1, 0, 0))),                    # B alone
            (193, 129, 65, False, dict(misalign=1, batch=2)),                  # a whole step and one k
            (135, 131, 129, False, dict(misalign=3, pad=(2, 4, 1, 0))),
            (2049, 1543, 129, True, dict(misalign=1)),                         # large tiles, eight waves
            (2049, 1543, 65, True, dict(misalign=1)),
            (2056, 1537, 200, True, dict()),
            (2056, 2184, 193, True, dict(pad=(1, 3, 0, 0))),                   # more tiles than CUs: eight waves where both have odd rows (A stored K x M)
            (2056, 2184, 200, True, dict(pad=(1, 3, 0, 0))),                   # in every storage
            (2056, 2184, 192, True, dict(pad=(1, 4, 0, 0))),                   # four where one alone has
            (2056, 2184, 128, True, dict(misalign=1))]:
        for out in ("f32", "bf16"):
            plain = out == "f32" and not (transA or transB)
            both_kernels(lambda: run_fused_case(oracle, M, N, K, transA=transA, transB=transB, act="relu", out=out, plan="direct", seed=M + K, **kw)[3].replace("_nn", "").replace(
                "_nt", "").replace("_tn", "").replace("_tt", ""), f"bf16_{'' if plain else 'fused_'}ragged_{tile[large]}x64", small=not large and (out == "bf16" or K <= 256 or K > 320))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(129, 127, 65), (33, 33, 4096), (1025, 9, 129), (9, 1999, 67), (1023, 515, 9), (77, 99, 700)])
def test_small_products(oracle, M, N, K):
    for dtype_kw in [dict(), dict(misalign=1)]:
        both_kernels(lambda: run_case(oracle, "bf16", M, N, K, alpha=0.5, act="gelu_tanh", seed=M + N + K, **dtype_kw)[3].replace("_splitk", ""), "bf16_ragged_64x64x64",
                     small=64 < K < 4096)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,tile", [(1405, 1501, 257, "128x128"), (1405, 1501, 256, "64x64"), (1401, 1401, 300, "64x64"), (1409, 1409, 300, "128x128")])
def test_large_tiles_for_more_than_two_rounds_of_small_ones(oracle, M, N, K, tile):
    _, _, _, cfg = run_case(oracle, "bf16", M, N, K, alpha=0.5, act="relu", seed=M + K)
    assert cfg == f"bf16_ragged_{tile}x64", cfg


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("K", [8, 9, 31, 33, 63, 64])
def test_one_step(oracle, transA, transB, K):
    """K of one step: read once, pulled back at its end, on both tiles and from odd elements."""
    for M, N, tile, kw in [(257, 1031, "64x64", dict(batch=3)), (259, 1024, "64x64", dict(misalign=1, batch=3)), (2056, 2189, "128x128", dict(misalign=1)),
                           (2056, 2184, "128x128", dict(pad=(1, 2, 0, 0)))]:
        for out in ("f32", "bf16"):
            _, _, _, cfg = run_fused_case(oracle, M, N, K, transA=transA, transB=transB, act="relu", out=out, plan="direct", seed=M + K, **kw)
            assert f"ragged_{tile}x64" in cfg, cfg


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,batch,kernel", [
    (5, 67, 31, 512, "bf16_generic_64x64x32"),               # 1024 tiles, hardly any of them inside
    (5, 67, 33, 512, "bf16_ragged_64x64x64"),                # more than one of the guarded kernel's steps
    (5, 67, 31, 511, "bf16_ragged_64x64x64"),                # fewer tiles
    (5, 67, 65, 512, "bf16_generic_64x64x32"),               # a few k past a 64-k step
    (5, 67, 73, 512, "bf16_ragged_64x64x64"),
    (5, 67, 65, 1024, "bf16_ragged_64x64x64"),               # more than 2^24 multiply-adds
    (11, 63, 31, 1024, "bf16_ragged_64x64x64"),              # more than one output in twelve inside
])
def test_slivers(oracle, M, N, K, batch, kernel):
    _, _, _, cfg = run_case(oracle, "bf16", M, N, K, batch=batch, alpha=0.5, act="relu", seed=M + K)
    assert cfg == kernel, cfg
