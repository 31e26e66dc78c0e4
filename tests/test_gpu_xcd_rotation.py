"""K walked from another tile on each XCD: K tiles a multiple of eight or not, one that K ends in, slices."""
import numpy as np
import pytest

import peak_inputs as pi

pytestmark = pytest.mark.gpu

TILES = ["m256x256w4a3", "m256x128w4a3", "m128x128w4a3", "m128x128w4a5", "m128x128k128w4a3", "m128x64q3"]


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from tests import gpu_util
    return gpu_util


def _variant(gu, name):
    return [gu.pg.peak_gemm_variant_name(i) for i in range(gu.pg.peak_gemm_variant_count())].index(name)


def _ints(dtype, transA, transB, M, N, K, seed):
    la, lb = pi.small_int_matrix(seed, 0, M, K, -2, 2, dtype), pi.small_int_matrix(seed, 1, K, N, -2, 2, dtype)
    return pi.store(la, bool(transA)), pi.store(lb, bool(transB))


# K tiles a multiple of eight or not, one that K ends in, in two slices
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dtype,transA", [(pi.BF16, 0), (pi.F16, 1)])
@pytest.mark.parametrize("K,split", [(4096, 1), (4168, 1), (8856, 2), (8200, 1)])
def test_k_from_another_tile_on_each_xcd(gu, oracle, tile, dtype, transA, K, split):
    pg = gu.pg
    M, N = 264, 1096                                        # workgroups on every XCD
    vid = _variant(gu, "%s_%s_%s" % (pi.DTYPE_NAMES[dtype], tile, "tt" if transA else "nt"))
    A, B = _ints(dtype, transA, 1, M, N, K, 8400)
    rows = [0, 1, 127, 128, 255, 256, 263]
    ref = oracle.gemm(dtype, transA, 1, M, N, K, 1.0, A, B, 0.0, None, rows=rows)
    got, _, info = gu.run_gemm(dtype, transA, 1, M, N, K, 1.0, 0.0, A, B, gu.nan_fill(M, N, pi.F32), flags=pg.force_flags(variant=vid, split=split), cdtype=pi.F32)
    assert np.array_equal(got[rows], ref), info             # small integers: exact in fp32 in any order
