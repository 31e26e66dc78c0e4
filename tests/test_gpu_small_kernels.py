"""The launches around the product: the ordered sum of the K slices where N ends inside a group of four columns, and the
transposition of an A stored K x M for the streaming kernels."""
import numpy as np
import pytest

import peak_inputs as pi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from tests import gpu_util
    return gpu_util


def _check(gu, oracle, dtype, ta, tb, M, N, K, flags, want):
    A, B = (pi.store(pi.logical_matrix(70, i, *s, "uniform", 1.0, dtype), bool(t))
            for i, (s, t) in enumerate((((M, K), ta), ((K, N), tb))))
    C = pi.store(pi.logical_matrix(70, 2, M, N, "uniform", 1.0, dtype), False)
    got, raw, info = gu.run_gemm(dtype, ta, tb, M, N, K, 0.5, 2.0, A, B, C, flags=flags)
    assert want in info, info
    gu.check_against_oracle(oracle, got, dtype, ta, tb, M, N, K, 0.5, A, B, 2.0, C, what=info)


@pytest.mark.parametrize("dtype", [pi.F32, pi.BF16])
@pytest.mark.parametrize("N", [1, 2, 3, 5, 127, 129, 130, 131, 132])
def test_sum_of_slices_ragged_columns(gu, oracle, dtype, N):
    for M, split in ((9, 2), (70, 7)):                        # fewer slices than are loaded at a time, and a remainder
        vid = next(i for i, n in gu.variants_for(dtype, 0, 1) if "_r64x64" in n)
        _check(gu, oracle, dtype, 0, 1, M, N, 7 * 128, gu.pg.force_flags(vid, split), "split=%d " % split)


@pytest.mark.parametrize("dtype,tb,M,K", [(pi.BF16, 1, 1, 4096), (pi.F16, 1, 64, 2048 + 128), (pi.BF16, 0, 37, 4096 + 64),
                                          (pi.F32, 0, 17, 2048 + 32), (pi.F32, 1, 63, 2048), (pi.F32, 0, 4, 2048), (pi.BF16, 1, 5, 2048), (pi.F16, 0, 16, 2048)])
def test_transposed_copy_of_a(gu, oracle, dtype, tb, M, K):
    pre, suf = {pi.F32: "f32", pi.F16: "f16", pi.BF16: "bf16"}[dtype], "_nt" if tb else "_nn"
    pg = gu.pg
    ran = 0
    for i in range(pg.peak_gemm_variant_count()):             # every streaming kernel that takes the shape
        n = pg.peak_gemm_variant_name(i)
        if not (n.startswith(pre + "_skinny") and n.endswith(suf)):
            continue
        try:
            pg.Plan(M, 264, K, dtype, 1, tb, flags=pg.force_flags(i)).close()
        except pg.PeakError as e:                             # more rows than the kernel has, a K that is no whole number of its stages
            assert e.status == pg.PEAK_ERR_UNSUPPORTED
            continue
        print(n, flush=True)
        _check(gu, oracle, dtype, 1, tb, M, 264, K, pg.force_flags(i), "acopy=1")
        ran += 1
    assert ran > 0


@pytest.mark.parametrize("dtype,name", [(pi.BF16, "_m256x128w4a3_nn"), (pi.BF16, "_m64x64q3_nn"), (pi.F16, "_t128x128w4_nn"),
                                        (pi.F32, "_r32x32_nn"), (pi.F32, "_m64x64q3_nn")])
@pytest.mark.parametrize("tiles_n,split", [(1, 2), (1, 7), (3, 3), (5, 2), (7, 9)])
def test_order_of_tiles_and_slices(gu, oracle, dtype, name, tiles_n, split):
    """Tiles x slices below, at odd distances from and above the 8 XCDs that share them out."""
    vid, full = next((i, n) for i, n in gu.variants_for(dtype, 0, 0) if n.endswith(name))
    N = {"m256x128w4a3": 128, "t128x128w4": 128, "r32x32": 32, "m64x64q3": 64}[name.split("_")[1]] * tiles_n - 8
    _check(gu, oracle, dtype, 0, 0, 24, N, split * 128, gu.pg.force_flags(vid, split), "split=%d " % split)


@pytest.mark.parametrize("dtype,rem", [(pi.F32, r) for r in (1, 2, 3)] + [(pi.BF16, r) for r in range(1, 8)])
@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0)])
def test_aligned_copies_of_rows_that_end_inside_a_chunk(gu, oracle, dtype, rem, ta, tb):
    """Every number of elements over, along K and along the matrices' other sides."""
    M, N, K = 2048 + rem, 2040 + rem, 1024 + rem
    A, B = (pi.store(pi.logical_matrix(71, i, *s, "uniform", 1.0, dtype), bool(t))
            for i, (s, t) in enumerate((((M, K), ta), ((K, N), tb))))
    C = pi.store(pi.logical_matrix(71, 2, M, N, "uniform", 1.0, dtype), False)
    got, raw, info = gu.run_gemm(dtype, ta, tb, M, N, K, 0.5, 2.0, A, B, C)
    assert "pack=3" in info, info
    gu.check_against_oracle(oracle, got, dtype, ta, tb, M, N, K, 0.5, A, B, 2.0, C, rows=[0, 1, 255, 1000, M - 9, M - 2, M - 1], what=info)
