"""Ways out of the 16-bit kernels that go straight through: the fused step on the accumulators, fp32 C and K slices, with tiles
that rows and columns of C end in."""
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


# a whole tile, edges inside a wave's rows and columns, N a whole number of 16-byte pieces or not, one row and column past a tile
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dtype,transA,transB", [(pi.BF16, 0, 1), (pi.F16, 1, 0)])
def test_fused_step_exact(gu, oracle, tile, dtype, transA, transB):
    pg = gu.pg
    vid = _variant(gu, "%s_%s_%s" % (pi.DTYPE_NAMES[dtype], tile, "tn" if transA else "nt"))
    for case, (M, N) in enumerate([(256, 256), (264, 520), (136, 72), (512, 8), (128, 136)] + ([(257, 257), (131, 387), (40, 515)] if not transA else [])):
        K = 64
        A, B = _ints(dtype, transA, transB, M, N, K, 8000 + case)
        ref0 = oracle.gemm(dtype, transA, transB, M, N, K, -1.0, A, B, 0.0, None)
        for kind in (pg.PEAK_BIAS_NONE, pg.PEAK_BIAS_PER_COLUMN, pg.PEAK_BIAS_PER_ROW):
            bias = None if kind == pg.PEAK_BIAS_NONE else pi.bias_vector(8100 + case, N if kind == pg.PEAK_BIAS_PER_COLUMN else M, ints=True)
            for act in (pg.PEAK_ACT_NONE, pg.PEAK_ACT_RELU, pg.PEAK_ACT_GELU_TANH):
                ref = oracle.bias_act(ref0, M, kind, bias, act)
                got, raw, info = gu.run_gemm(dtype, transA, transB, M, N, K, -1.0, 0.0, A, B, gu.nan_fill(M, N + 8, dtype),
                                             flags=pg.force_flags(variant=vid, split=1), fused=(kind, bias, act))
                if act == pg.PEAK_ACT_GELU_TANH:            # one rounding to storage and a few units of fp32 on either side of it
                    bound = gu.U_OUT[dtype] * np.abs(ref) + 2.0 ** -20 * (1.0 + np.abs(ref)) + (2.0 ** -24 if dtype == pi.F16 else 0.0)
                    assert np.all(np.abs(got - ref) <= bound), (info, M, N, kind, act)
                else:
                    assert np.array_equal(got, ref), (info, M, N, kind, act)
                assert np.array_equal(raw[:, N:], gu.nan_fill(M, 8, dtype)), (info, M, N, kind, act)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dtype,transA,transB", [(pi.BF16, 0, 1), (pi.F16, 1, 0)])
def test_fp32_c_and_slices_exact(gu, oracle, tile, dtype, transA, transB):
    pg = gu.pg
    vid = _variant(gu, "%s_%s_%s" % (pi.DTYPE_NAMES[dtype], tile, "tn" if transA else "nt"))
    K = 512
    for case, (M, N) in enumerate([(256, 256), (264, 520), (136, 72), (128, 136)] + ([(257, 260), (131, 388), (259, 261)] if not transA else [])):
        A, B = _ints(dtype, transA, transB, M, N, K, 8200 + case)
        C = pi.store(pi.small_int_matrix(8300 + case, 2, M, N, -3, 3, pi.F32), False, N + 4)
        for alpha, beta, split, cdtype in [(1.0, 0.0, 1, pi.F32), (-2.0, 1.0, 1, pi.F32), (1.0, -0.5, 1, pi.F32), (1.0, 2.0, 3, pi.F32), (1.0, 0.0, 2, dtype)]:
            C0 = C if beta != 0 else gu.nan_fill(M, N + 4, cdtype)
            ref = oracle.gemm(dtype, transA, transB, M, N, K, alpha, A, B, beta, C if beta != 0 else None, **({"cdtype": pi.F32} if beta != 0 else {}))
            got, raw, info = gu.run_gemm(dtype, transA, transB, M, N, K, alpha, beta, A, B, C0,
                                         flags=pg.force_flags(variant=vid, split=split), cdtype=cdtype)
            if cdtype == pi.F32:
                assert np.array_equal(got, ref), (info, M, N, alpha, beta, split)
            else:
                assert np.all(np.abs(got - ref) <= gu.U_OUT[dtype] * np.abs(ref)), (info, M, N, split)
            assert np.array_equal(raw[:, N:].view(np.uint8), C0[:, N:].view(np.uint8)), (info, M, N, alpha, beta, split)


# C_in and a C of the operands' type: whole tiles, which go straight through, and edges, with rows of C on 16 bytes, 2, 6 and 12 off
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dtype,transA,transB", [(pi.BF16, 0, 1), (pi.F16, 1, 0)])
def test_16_bit_c_with_c_in_exact(gu, oracle, tile, dtype, transA, transB):
    pg = gu.pg
    vid = _variant(gu, "%s_%s_%s" % (pi.DTYPE_NAMES[dtype], tile, "tn" if transA else "nt"))
    K = 64
    for case, (M, N) in enumerate([(256, 256), (512, 768), (264, 520), (136, 72)]):
        A, B = _ints(dtype, transA, transB, M, N, K, 8600 + case)
        for pad, alpha, beta in [(0, 1.0, 1.0), (1, -1.0, 2.0), (3, 0.5, -1.0), (6, 1.0, 0.5)]:
            C = pi.store(pi.small_int_matrix(8700 + case, 2, M, N, -8, 8, dtype), False, N + pad)
            ref = oracle.gemm(dtype, transA, transB, M, N, K, alpha, A, B, beta, C)       # multiples of 0.5 below 512: exact in fp32
            got, raw, info = gu.run_gemm(dtype, transA, transB, M, N, K, alpha, beta, A, B, C, flags=pg.force_flags(variant=vid, split=1))
            assert np.all(np.abs(got - ref) <= gu.U_OUT[dtype] * np.abs(ref)), (info, M, N, pad, alpha, beta)
            assert np.array_equal(raw[:, N:], C[:, N:]), (info, M, N, pad)
