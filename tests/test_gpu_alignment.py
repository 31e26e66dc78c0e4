"""Operands of any alignment: blocks of larger matrices that start one element in, with odd leading dimensions and
NaN in everything around the block, through every register-staged ("_r") kernel, at the edges of its 16-byte chunks,
K tiles and tiles, unsplit and split.  A chunk fetched beyond the block, or shifted into the wrong place, brings a NaN
or a wrong product into the result."""
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


def _block(gu, values, pad, off, dtype):
    """(flat buffer, leading dimension): `values` as a block of a NaN-filled buffer, `off` elements in."""
    rows, cols = values.shape
    buf = gu.nan_fill(1, off + rows * (cols + pad), dtype).ravel()
    buf[off:].reshape(rows, cols + pad)[:, :cols] = values
    return buf, cols + pad


@pytest.mark.parametrize("dtype", [pi.F32, pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
def test_blocks_at_odd_addresses(gu, oracle, dtype, transA, transB):
    import torch
    es = pi.DTYPE_SIZE[dtype]
    epc, bk = 16 // es, 128 // es
    shapes = [(67, 71, 4 * bk + 1, 2), (130, 66, 2 * bk - 1, None), (33, 2 * epc + 1, epc, None), (epc - 1, 65, epc + 1, None),
              (64, epc - 1, 3 * bk + epc - 1, 3), (5, 3, epc - 1, None)]
    for vid, name in gu.variants_for(dtype, transA, transB):
        if "_r" not in name:
            continue
        for case, (M, N, K, split) in enumerate(shapes):
            la = pi.logical_matrix(50 + case, 0, M, K, "uniform", 1.0, dtype)
            lb = pi.logical_matrix(50 + case, 1, K, N, "uniform", 1.0, dtype)
            lc = pi.logical_matrix(50 + case, 2, M, N, "uniform", 1.0, dtype)
            A, B = pi.store(la, bool(transA)), pi.store(lb, bool(transB))
            pad, off = 1 + case % 2, 1 + case % 3
            (bufA, lda), (bufB, ldb), (bufC, ldc) = (_block(gu, x, pad, off, dtype) for x in (A, B, lc))
            dA, dB, dC = gu.to_dev(bufA), gu.to_dev(bufB), gu.to_dev(bufC)
            print(name, M, N, K, split, flush=True)
            with gu.pg.Plan(M, N, K, dtype, transA, transB, lda, ldb, ldc, gu.pg.force_flags(vid, split)) as plan:
                ws = torch.empty(max(plan.workspace_bytes, 256), dtype=torch.uint8, device="cuda")
                plan.run(0.5, dA.data_ptr() + off * es, dB.data_ptr() + off * es, 2.0, dC.data_ptr() + off * es,
                         ws.data_ptr(), plan.workspace_bytes, torch.cuda.current_stream().cuda_stream)
                torch.cuda.synchronize()
            out = gu.from_dev(dC, dtype)
            block = out[off:].reshape(M, ldc)
            got = pi.to_f64(np.ascontiguousarray(block[:, :N]), dtype)
            gu.check_against_oracle(oracle, got, dtype, transA, transB, M, N, K, 0.5, A, B, 2.0, lc, what=(name, M, N, K, split))
            # nothing outside the block was written
            assert np.array_equal(out[:off].view(np.uint8), bufC[:off].view(np.uint8))
            assert np.array_equal(block[:, N:].view(np.uint8), bufC[off:].reshape(M, ldc)[:, N:].view(np.uint8))
