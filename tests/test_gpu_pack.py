"""Plans that write aligned copies of their operands first ("pack=" in the plan description): odd sizes and leading
dimensions, blocks of NaN-filled larger matrices at odd addresses, one operand aligned and the other not, all layouts;
copies behind the partials of a K split and of a cut last round; a run without room for the copies, and the entry point
with the fixed array where they outgrow it, takes the stand-in for any alignment."""
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
    for s, b in [((2049, 2047, 1031), (1, 1)), ((2056, 2048, 1024), (3, 0)), ((2056, 2048, 1024), (0, 3))]])
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
        assert pack == (3 if K % 8 else (1 if blocks[0] else 0) | (2 if blocks[1] else 0)) and "_r" in re.search(r"unaligned=(\S+)", info).group(1), info
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


def _product(gu, dtype, transA, transB, M, N, K, seed):
    """Stored whole matrices of a product on the host, their device copies, and C full of NaN."""
    A, B = (pi.store(pi.logical_matrix(seed, i, *s, "uniform", 1.0, dtype), bool(t)) for i, (s, t) in enumerate((((M, K), transA), ((K, N), transB))))
    return A, B, gu.to_dev(A), gu.to_dev(B), gu.to_dev(gu.nan_fill(M, N, dtype))


def _check(gu, oracle, dC, dtype, transA, transB, M, N, K, A, B, what):
    import torch
    torch.cuda.synchronize()
    rows = sorted({0, 1, 127, 128, 255, 256, 511, M // 2, M - 130, M - 9, M - 2, M - 1} & set(range(M)))
    got = pi.to_f64(gu.from_dev(dC, dtype), dtype)
    gu.check_against_oracle(oracle, got, dtype, transA, transB, M, N, K, 1.0, A, B, 0.0, None, rows=rows, what=what)


@pytest.mark.parametrize("dtype,transA,transB,M,N,K,streamk", [
    (pi.F32, 1, 0, 759, 1437, 853, False), (pi.F16, 0, 0, 1353, 747, 3209, False), (pi.BF16, 1, 1, 811, 1383, 3221, False),
    (pi.F16, 0, 1, 3497, 4657, 611, True), (pi.BF16, 1, 1, 4263, 3875, 801, True)])
def test_copies_behind_partials(gu, oracle, dtype, transA, transB, M, N, K, streamk):
    import torch
    A, B, dA, dB, dC = _product(gu, dtype, transA, transB, M, N, K, 41)
    with gu.pg.Plan(M, N, K, dtype, transA, transB) as plan:
        info = plan.info()
        fields = dict(w.split("=", 1) for w in info.split() if "=" in w)
        assert fields["pack"] == "3" and int(fields["split"]) > 1 and (fields["streamk"] != "0") == streamk, info
        ws = torch.full((plan.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")       # NaN wherever nothing is written
        plan.run(1.0, dA.data_ptr(), dB.data_ptr(), 0.0, dC.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        _check(gu, oracle, dC, dtype, transA, transB, M, N, K, A, B, info)


# (products of more tiles than the stand-in splits K for: it needs no workspace and writes nothing to the one it is given)
@pytest.mark.parametrize("dtype,transA,transB,M,N,K", [
    (dt, ta, tb, 2049, 2047, 1031) for dt in (pi.F32, pi.BF16) for ta, tb in itertools.product([0, 1], [0, 1])] + [(pi.F16, 0, 1, 4097, 4099, 515)])
def test_workspace_without_room_for_the_copies_takes_the_stand_in(gu, oracle, dtype, transA, transB, M, N, K):
    import torch
    A, B, dA, dB, dC = _product(gu, dtype, transA, transB, M, N, K, 42)
    stream = torch.cuda.current_stream().cuda_stream
    with gu.pg.Plan(M, N, K, dtype, transA, transB) as plan:
        assert "pack=3" in plan.info() and plan.workspace_bytes > 0, plan.info()
        ws = torch.full((plan.workspace_bytes + 16,), 0xA5, dtype=torch.uint8, device="cuda")
        # one byte short, off 256 bytes, none at all
        for ptr, nbytes in ((ws.data_ptr(), plan.workspace_bytes - 1), (ws.data_ptr() + 16, plan.workspace_bytes), (0, 0)):
            dC.copy_(gu.to_dev(gu.nan_fill(M, N, dtype)))
            plan.run(1.0, dA.data_ptr(), dB.data_ptr(), 0.0, dC.data_ptr(), ptr, nbytes, stream)
            _check(gu, oracle, dC, dtype, transA, transB, M, N, K, A, B, (plan.info(), nbytes))
        assert bool((ws == 0xA5).all())                          # no copies were made
        plan.run(1.0, dA.data_ptr(), dB.data_ptr(), 0.0, dC.data_ptr(), ws.data_ptr(), plan.workspace_bytes, stream)
        assert not bool((ws == 0xA5).all())


@pytest.mark.parametrize("dtype,transA,transB,M,N,K", [(pi.BF16, 0, 1, 4097, 4099, 2051), (pi.F32, 1, 0, 2049, 3001, 2051)])
def test_copies_larger_than_the_fixed_array_take_the_stand_in(gu, oracle, dtype, transA, transB, M, N, K):
    import torch
    A, B, dA, dB, dC = _product(gu, dtype, transA, transB, M, N, K, 43)
    with gu.pg.Plan(M, N, K, dtype, transA, transB) as plan:
        assert "pack=3" in plan.info() and plan.workspace_bytes > gu.pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES, plan.info()
        assert gu.pg.peak_gemm_run_static(plan.handle, 1.0, dA.data_ptr(), dB.data_ptr(), 0.0, dC.data_ptr(),
                                          torch.cuda.current_stream().cuda_stream) == gu.pg.PEAK_OK
        _check(gu, oracle, dC, dtype, transA, transB, M, N, K, A, B, plan.info())


@pytest.mark.parametrize("dtype", [pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
@pytest.mark.parametrize("rem", [2, 4, 6])
def test_copies_only_against_rows_on_odd_addresses(gu, oracle, dtype, transA, transB, rem):
    """Even leading dimensions: copies where a base puts every row on odd 2-byte addresses, none where both are even."""
    import torch
    M, N, K = 2048 + rem, 2040 + rem, 1024 + rem
    A, B = (pi.store(pi.logical_matrix(44, i, *s, "uniform", 1.0, dtype), bool(t)) for i, (s, t) in enumerate((((M, K), transA), ((K, N), transB))))
    stream = torch.cuda.current_stream().cuda_stream
    with gu.pg.Plan(M, N, K, dtype, transA, transB) as plan:
        assert "pack=3" in plan.info() and "oddbase=1" in plan.info(), plan.info()
        for offs in ((0, 0), (1, 0), (0, 1), (1, 1), (2, 2)):
            dA, dB = (gu.to_dev(_block(gu, x, 0, o, dtype)[0]) for x, o in zip((A, B), offs))
            dC = gu.to_dev(gu.nan_fill(M, N, dtype))
            ws = torch.full((plan.workspace_bytes,), 0xA5, dtype=torch.uint8, device="cuda")
            plan.run(1.0, dA.data_ptr() + 2 * offs[0], dB.data_ptr() + 2 * offs[1], 0.0, dC.data_ptr(), ws.data_ptr(), ws.numel(), stream)
            _check(gu, oracle, dC, dtype, transA, transB, M, N, K, A, B, (plan.info(), offs))
            assert bool((ws == 0xA5).all()) == (offs[0] % 2 == 0 and offs[1] % 2 == 0), offs


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
