"""Plans that write aligned copies of their operands first ("pack=" in the plan description): odd sizes and leading
dimensions, blocks of NaN-filled larger matrices at odd addresses, one operand aligned and the other not, all layouts;
a run without room for the copies takes the register-staged stand-in, and so does the entry point with the fixed array."""
import itertools
import re

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


def _block(gu, values, pad, off, dtype):
    rows, cols = values.shape
    buf = gu.nan_fill(1, off + rows * (cols + pad), dtype).ravel()
    buf[off:].reshape(rows, cols + pad)[:, :cols] = values
    return buf, cols + pad


@pytest.mark.parametrize("dtype,transA,transB,sizes,blocks", [
    (dt, ta, tb, s, b) for dt in (pi.F32, pi.BF16, pi.F16) for ta, tb in itertools.product([0, 1], [0, 1])
    for s, b in [((2049, 2047, 1031), (1, 1)), ((2056, 2048, 1024), (3, 0))]])
def test_aligned_copies(gu, oracle, dtype, transA, transB, sizes, blocks):
    import torch
    pg = gu.pg
    M, N, K = sizes
    es = pi.DTYPE_SIZE[dtype]
    la, lb = (pi.logical_matrix(40, i, *s, "uniform", 1.0, dtype) for i, s in enumerate(((M, K), (K, N))))
    lc = pi.logical_matrix(40, 2, M, N, "uniform", 1.0, dtype)
    A, B = pi.store(la, bool(transA)), pi.store(lb, bool(transB))
    bufA, lda = _block(gu, A, blocks[0], blocks[0], dtype)
    bufB, ldb = _block(gu, B, blocks[1], blocks[1], dtype)
    dA, dB = gu.to_dev(bufA), gu.to_dev(bufB)
    rows = sorted({0, 1, 31, 127, 128, 255, 256, 1000, M // 2, M - 9, M - 8, M - 2, M - 1})
    stream = torch.cuda.current_stream().cuda_stream
    with pg.Plan(M, N, K, dtype, transA, transB, lda, ldb, N) as plan:
        info = plan.info()
        pack = int(re.search(r"pack=(\d)", info).group(1))
        assert pack == (3 if blocks[1] else 1) and "_r" in re.search(r"unaligned=(\S+)", info).group(1), info
        args = (0.5, dA.data_ptr() + blocks[0] * es, dB.data_ptr() + blocks[1] * es, 2.0)
        for nbytes in (plan.workspace_bytes, pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES, None):
            dC = gu.to_dev(lc)
            if nbytes is None:
                assert pg.peak_gemm_run_static(plan.handle, *args, dC.data_ptr(), stream) == pg.PEAK_OK
            else:
                ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")     # NaN wherever nothing is written
                plan.run(*args, dC.data_ptr(), ws.data_ptr(), nbytes, stream)
            torch.cuda.synchronize()
            got = pi.to_f64(gu.from_dev(dC, dtype), dtype)
            gu.check_against_oracle(oracle, got, dtype, transA, transB, M, N, K, 0.5, A, B, 2.0, lc, rows=rows, what=(info, nbytes))


def test_workspace_off_256_bytes_takes_the_stand_in(gu):
    import torch
    pg = gu.pg
    M, N, K = 4097, 4099, 515                                   # more tiles than the stand-in ever splits K for
    A, B = (torch.randn(r, K, device="cuda", dtype=torch.bfloat16) for r in (M, N))
    stream = torch.cuda.current_stream().cuda_stream
    with pg.Plan(M, N, K, pi.BF16, 0, 1, K, K, N) as plan:
        assert "pack=3" in plan.info(), plan.info()
        ws = torch.empty(plan.workspace_bytes + 16, dtype=torch.uint8, device="cuda")
        out = []
        for ptr, nbytes in ((ws.data_ptr() + 16, plan.workspace_bytes), (0, 0)):
            C = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
            plan.run(1.0, A.data_ptr(), B.data_ptr(), 0.0, C.data_ptr(), ptr, nbytes, stream)
            torch.cuda.synchronize()
            out.append(C)
    assert torch.equal(out[0], out[1])                           # (NaN would not compare equal)


@pytest.mark.parametrize("static", [0, 1])
def test_aligned_copies_under_capture(gu, static):
    """Replays copy what the operands hold then, not what they held at capture."""
    import torch
    pg = gu.pg
    M, N, K = 2049, 2047, 1031
    A, B = (torch.randn(r, K, device="cuda", dtype=torch.bfloat16) for r in (M, N))
    C, E = (torch.zeros(M, N, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    with pg.Plan(M, N, K, pi.BF16, 0, 1, K, K, N) as plan:
        assert "pack=3" in plan.info(), plan.info()
        ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")

        def run(out):
            stream = torch.cuda.current_stream().cuda_stream
            if static:
                assert pg.peak_gemm_run_static(plan.handle, 1.0, A.data_ptr(), B.data_ptr(), 0.0, out.data_ptr(), stream) == pg.PEAK_OK
            else:
                plan.run(1.0, A.data_ptr(), B.data_ptr(), 0.0, out.data_ptr(), ws.data_ptr(), ws.numel(), stream)

        run(E)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run(C)
        for _ in range(3):
            A.copy_(torch.randn(M, K, device="cuda"))
            run(E)
            torch.cuda.synchronize()
            C.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(C, E)
