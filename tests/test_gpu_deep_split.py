"""Deep K split with its stand-in: whole workspace, one byte short, off its boundary, none, and the entry point with the fixed array."""
import pytest
import numpy as np

import peak_inputs as pi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from tests import gpu_util
    return gpu_util


# rows and columns that end inside a tile, K inside a K tile, the last slice shorter; whether the stand-in splits K itself
@pytest.mark.parametrize("dtype,transA,transB,M,N,K,splits", [
    (pi.BF16, 0, 0, 391, 5504, 11392, False), (pi.F16, 0, 1, 340, 3700, 15152, True), (pi.BF16, 1, 0, 640, 4160, 11072, False),
    (pi.F16, 1, 1, 568, 3012, 19432, True)])
def test_deep_split_and_its_stand_in(gu, oracle, dtype, transA, transB, M, N, K, splits):
    import torch
    pg = gu.pg
    g = np.random.default_rng(45)
    bits = lambda r, c: (torch.from_numpy(g.uniform(-1, 1, (r, c)).astype(np.float32))
                         .to(torch.bfloat16 if dtype == pi.BF16 else torch.float16).view(torch.int16).numpy().view(np.uint16))
    A, B = bits(*((K, M) if transA else (M, K))), bits(*((N, K) if transB else (K, N)))
    dA, dB = gu.to_dev(A), gu.to_dev(B)
    rows = sorted({0, 1, 127, 255, 256, 263, M - 9, M - 1} & set(range(M)))
    ref, bound = gu.elementwise_bound(oracle, dtype, transA, transB, M, N, K, 1.0, A, B, 0.0, None, rows)
    stream = torch.cuda.current_stream().cuda_stream
    with pg.Plan(M, N, K, dtype, transA, transB) as plan:
        info, need = plan.info(), plan.workspace_bytes
        assert "small=none" not in info and need > pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES, info
        ws = torch.full((need + 16,), 0xFF, dtype=torch.uint8, device="cuda")                 # NaN wherever nothing is written
        seen = []
        # whole, one byte short, as large as the fixed array, the entry point with that array; off its boundary, none
        for at, nbytes, status in ((0, need, pg.PEAK_OK), (0, need - 1, pg.PEAK_OK), (0, pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES, pg.PEAK_OK),
                                   (None, None, pg.PEAK_OK), (16, need, pg.PEAK_ERR_INVALID_ARG if splits else pg.PEAK_OK),
                                   (None, 0, pg.PEAK_ERR_WORKSPACE if splits else pg.PEAK_OK)):
            dC = gu.to_dev(gu.nan_fill(M, N, dtype))
            args = (plan.handle, 1.0, dA.data_ptr(), dB.data_ptr(), 0.0, dC.data_ptr())
            ptr = 0 if at is None else ws.data_ptr() + at
            got = pg.peak_gemm_run_static(*args, stream) if nbytes is None else pg.peak_gemm_run(*args, ptr, nbytes, stream)
            assert got == status, (info, at, nbytes, got)
            torch.cuda.synchronize()
            got = gu.from_dev(dC, dtype)
            if status != pg.PEAK_OK:                                                          # refused: nothing launched
                assert np.array_equal(got, gu.nan_fill(M, N, dtype)), (info, at, nbytes)
                continue
            gu.assert_elementwise(pi.to_f64(got, dtype)[rows], ref, bound, (info, at, nbytes))
            seen.append(got)
        # the stand-in's bits whatever the smaller workspace
        assert len(seen) == (4 if splits else 6)
        assert all((x == seen[1]).all() for x in seen[2:])
