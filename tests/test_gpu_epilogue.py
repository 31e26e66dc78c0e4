"""The tiled kernels' way out with 16-byte stores, through every tiled variant: rows and columns that end inside a slab
of 32 rows and inside a tile, rows of C off 16 bytes, C_in, per-row and per-column bias with ReLU, an fp32 C of 16-bit
operands and split-K partials.  Integer data: every result is exact, so a value taken from the wrong row, column or
slab shows."""
import itertools

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


@pytest.mark.parametrize("dtype", [pi.F32, pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
def test_vector_epilogue_exact(gu, oracle, dtype, transA, transB):
    pg = gu.pg
    K = 64
    # (M, N, padding of C's rows, split, bias kind, fp32 C)
    cases = [(296, 264, 0, None, pg.PEAK_BIAS_PER_ROW, False), (256, 512, 1, None, pg.PEAK_BIAS_PER_COLUMN, False),
             (296, 328, 3, None, pg.PEAK_BIAS_PER_ROW, True), (264, 520, 0, 2, pg.PEAK_BIAS_PER_COLUMN, True)]
    data = {}
    for vid, name in gu.variants_for(dtype, transA, transB):
        if "skinny" in name:
            continue
        for case, (M, N, pad, split, kind, c_f32) in enumerate(cases):
            cdtype = pi.F32 if c_f32 else dtype
            if case not in data:
                A = pi.store(pi.small_int_matrix(70 + case, 0, M, K, -1, 1, dtype), bool(transA))
                B = pi.store(pi.small_int_matrix(70 + case, 1, K, N, -1, 1, dtype), bool(transB))
                C = pi.store(pi.small_int_matrix(70 + case, 2, M, N, -9, 9, cdtype), False, N + pad)
                bias = (np.arange(M if kind == pg.PEAK_BIAS_PER_ROW else N) % 13 - 6).astype(np.float32)
                ref = oracle.gemm(dtype, transA, transB, M, N, K, 1.0, A, B, 2.0, C, cdtype=cdtype)
                data[case] = A, B, C, bias, oracle.bias_act(ref, M, kind, bias, pg.PEAK_ACT_RELU)
            A, B, C, bias, ref = data[case]
            got, raw, info = gu.run_gemm(dtype, transA, transB, M, N, K, 1.0, 2.0, A, B, C,
                                         flags=pg.force_flags(vid, split), fused=(kind, bias, pg.PEAK_ACT_RELU),
                                         cdtype=cdtype)
            assert np.array_equal(got, ref), (name, case, info)
            assert np.array_equal(raw[:, N:].view(np.uint8), C[:, N:].view(np.uint8)), (name, case)


@pytest.mark.parametrize("dtype", [pi.F32, pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
def test_plain_edge_tiles_exact(gu, oracle, dtype, transA, transB):
    """beta = 0 and no fused step on tiles that C ends inside of, at whole 16-byte pieces: the same way out as interior
    tiles, by rows and columns.  What C holds before (NaN) reaches nothing, and nothing beyond M and N is written."""
    pg = gu.pg
    K = 64
    data = {}
    for vid, name in gu.variants_for(dtype, transA, transB):
        if "skinny" in name:
            continue
        for case, (M, N, pad, kind) in enumerate([(296, 264, 0, None), (72, 136, 1, None), (8, 8, 3, None), (264, 72, 2, pg.PEAK_BIAS_PER_COLUMN),
                                                  (40, 200, 1, pg.PEAK_BIAS_PER_ROW)]):
            if case not in data:
                A = pi.store(pi.small_int_matrix(60 + case, 0, M, K, -1, 1, dtype), bool(transA))
                B = pi.store(pi.small_int_matrix(60 + case, 1, K, N, -1, 1, dtype), bool(transB))
                C = gu.nan_fill(M + 1, N + pad, dtype)
                bias = (np.arange(M if kind == pg.PEAK_BIAS_PER_ROW else N) % 13 - 6).astype(np.float32)
                ref = oracle.gemm(dtype, transA, transB, M, N, K, 1.0, A, B, 0.0, None)
                data[case] = A, B, C, bias, ref if kind is None else oracle.bias_act(ref, M, kind, bias, pg.PEAK_ACT_NONE)
            A, B, C, bias, ref = data[case]
            got, raw, info = gu.run_gemm(dtype, transA, transB, M, N, K, 1.0, 0.0, A, B, C, flags=gu.pg.force_flags(vid, 1),
                                         fused=None if kind is None else (kind, bias, pg.PEAK_ACT_NONE))
            assert np.array_equal(got, ref), (name, case, info)
            assert np.array_equal(raw[:, N:].view(np.uint8), C[:, N:].view(np.uint8)), (name, case)
            assert np.array_equal(raw[M:].view(np.uint8), C[M:].view(np.uint8)), (name, case)


@pytest.mark.parametrize("dtype", [pi.F32, pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
def test_ragged_right_edge_exact(gu, oracle, dtype, transA, transB):
    """N that ends one to seven columns into a lane's piece, a wave tile or a tile: the last lane's overlapping store,
    and the columns that are fewer than a lane stores."""
    pg = gu.pg
    K = 64
    data = {}
    for vid, name in gu.variants_for(dtype, transA, transB):
        if "skinny" in name:
            continue
        for case, (M, N, split, c_f32) in enumerate([(72, 257, None, False), (40, 391, None, False), (264, 331, None, True),
                                                     (72, 133, 2, False), (33, 66, None, False)]):
            cdtype = pi.F32 if c_f32 else dtype
            if case not in data:
                A = pi.store(pi.small_int_matrix(80 + case, 0, M, K, -1, 1, dtype), bool(transA))
                B = pi.store(pi.small_int_matrix(80 + case, 1, K, N, -1, 1, dtype), bool(transB))
                C = pi.store(pi.small_int_matrix(80 + case, 2, M, N, -9, 9, cdtype), False, N + case % 3)
                bias = (np.arange(N) % 13 - 6).astype(np.float32)
                ref = oracle.gemm(dtype, transA, transB, M, N, K, 1.0, A, B, -1.0, C, cdtype=cdtype)
                data[case] = A, B, C, bias, oracle.bias_act(ref, M, pg.PEAK_BIAS_PER_COLUMN, bias, pg.PEAK_ACT_RELU)
            A, B, C, bias, ref = data[case]
            try:
                got, raw, info = gu.run_gemm(dtype, transA, transB, M, N, K, 1.0, -1.0, A, B, C,
                                             flags=pg.force_flags(vid, split),
                                             fused=(pg.PEAK_BIAS_PER_COLUMN, bias, pg.PEAK_ACT_RELU), cdtype=cdtype)
            except pg.PeakError as e:
                assert e.status == pg.PEAK_ERR_UNSUPPORTED        # rows that the direct copies do not take
                continue
            assert np.array_equal(got, ref), (name, case, info)
            assert np.array_equal(raw[:, N:].view(np.uint8), C[:, N:].view(np.uint8)), (name, case)
