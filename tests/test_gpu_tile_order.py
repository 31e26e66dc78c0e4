"""Tiles by the host's reciprocals: one tile, one row or column of them, bands cut by the last rows, primes, K slices."""
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


# (tile rows, tile columns) of 64 x 64 ring tiles, 256 x 256 tiles and streaming tiles, slices
@pytest.mark.parametrize("dtype,name,unit,grids", [
    (pi.BF16, "bf16_m64x64q3_nt", 64, [(1, 1, 1), (1, 13, 1), (13, 1, 1), (9, 7, 1), (17, 5, 3), (11, 23, 2), (4, 16, 1), (5, 17, 4)]),
    (pi.F16, "f16_m256x256w4a3_nt", 256, [(1, 1, 2), (3, 5, 1), (9, 2, 3), (5, 17, 1)]),
    (pi.F32, "f32_m32x32q3_nt", 32, [(1, 1, 1), (1, 13, 2), (19, 1, 1), (9, 7, 3), (17, 19, 1)])])
def test_every_tile_once(gu, oracle, dtype, name, unit, grids):
    pg = gu.pg
    vid = [pg.peak_gemm_variant_name(i) for i in range(pg.peak_gemm_variant_count())].index(name)
    for case, (tm, tn, split) in enumerate(grids):
        M, N, K = tm * unit - 5, tn * unit - 3, 512
        A = pi.store(pi.small_int_matrix(8500 + case, 0, M, K, -1, 1, dtype), False)
        B = pi.store(pi.small_int_matrix(8500 + case, 1, K, N, -1, 1, dtype), True)
        C0 = gu.nan_fill(M, N, pi.F32)
        got, _, info = gu.run_gemm(dtype, 0, 1, M, N, K, 1.0, 0.0, A, B, C0, flags=pg.force_flags(variant=vid, split=split), cdtype=pi.F32)
        want = pi.to_f64(A, dtype) @ pi.to_f64(B, dtype).T          # small integers: exact
        assert np.array_equal(got, want), (info, tm, tn, split)
