"""The small-tile ring kernels ("_m...q<stages>"): K shorter than the ring, a whole number of trips round it and one
tile more or less, K ending inside a tile, unsplit and split, with rows and columns that end inside a tile."""
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


@pytest.mark.parametrize("dtype", [pi.F32, pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
def test_ring_lengths(gu, oracle, dtype, transA, transB):
    es = pi.DTYPE_SIZE[dtype]
    epc = 16 // es
    seen = 0
    for vid, name in gu.variants_for(dtype, transA, transB):
        ring = re.search(r"_m\d+x\d+(k128)?q(\d)_", name)
        if not ring:
            continue
        seen += 1
        with gu.pg.Plan(64, 64, 4096, dtype, transA, transB, flags=gu.pg.force_flags(vid)) as p:
            bk = int(re.search(r"tile=\d+x\d+x(\d+)", p.info()).group(1))
        stages = int(ring.group(2))
        for case, (tiles, tail, split) in enumerate([(1, 0, None), (1, epc - bk, None), (stages - 1, epc, None), (stages, 0, None),
                                                      (stages + 1, epc - bk, None), (2 * stages, bk - epc, 3)]):
            M, N, K = 136 if transA else 129, 72 if not transB else 70, tiles * bk + tail
            A, B = (pi.store(pi.logical_matrix(90 + case, i, *s, "uniform", 1.0, dtype), bool(t))
                    for i, (s, t) in enumerate((((M, K), transA), ((K, N), transB))))
            C = pi.store(pi.logical_matrix(90 + case, 2, M, N, "uniform", 1.0, dtype), False)
            got, raw, info = gu.run_gemm(dtype, transA, transB, M, N, K, 0.5, 2.0, A, B, C, flags=gu.pg.force_flags(vid, split))
            gu.check_against_oracle(oracle, got, dtype, transA, transB, M, N, K, 0.5, A, B, 2.0, C, what=(info, K))
            got2, raw2, _ = gu.run_gemm(dtype, transA, transB, M, N, K, 0.5, 2.0, A, B, C, flags=gu.pg.force_flags(vid, split))
            assert np.array_equal(raw.view(np.uint8), raw2.view(np.uint8)), info
    assert seen >= 2
