"""The kernels for operands of any alignment ("_r"): K shorter than the ring of direct copies, whole trips round it and a tile more
or less, K ending inside a tile or on its end with the matrix edge inside a 16-byte chunk, rows on odd and even addresses, in blocks
of NaN-filled buffers; and leading dimensions beyond the copies' 32-bit offsets."""
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
    """(flat buffer, leading dimension): `values` as a block of a NaN-filled buffer that ends with its last element."""
    rows, cols = values.shape
    buf = gu.nan_fill(1, off + rows * (cols + pad), dtype).ravel()
    buf[off:].reshape(rows, cols + pad)[:, :cols] = values
    return buf[:buf.size - pad].copy(), cols + pad


def _run(gu, oracle, dtype, transA, transB, M, N, K, vid, split, pads, offs, what):
    import torch
    es = pi.DTYPE_SIZE[dtype]
    la, lb, lc = (pi.logical_matrix(60, i, *s, "uniform", 1.0, dtype) for i, s in enumerate(((M, K), (K, N), (M, N))))
    A, B = pi.store(la, bool(transA)), pi.store(lb, bool(transB))
    (bufA, lda), (bufB, ldb) = (_block(gu, x, p, o, dtype) for x, p, o in zip((A, B), pads, offs))
    dA, dB, dC = gu.to_dev(bufA), gu.to_dev(bufB), gu.to_dev(lc)
    print(what, M, N, K, split, pads, offs, flush=True)
    with gu.pg.Plan(M, N, K, dtype, transA, transB, lda, ldb, N, gu.pg.force_flags(vid, split)) as plan:
        ws = torch.empty(max(plan.workspace_bytes, 256), dtype=torch.uint8, device="cuda")
        plan.run(0.5, dA.data_ptr() + offs[0] * es, dB.data_ptr() + offs[1] * es, 2.0, dC.data_ptr(), ws.data_ptr(),
                 plan.workspace_bytes, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    got = pi.to_f64(np.ascontiguousarray(gu.from_dev(dC, dtype)), dtype)
    gu.check_against_oracle(oracle, got, dtype, transA, transB, M, N, K, 0.5, A, B, 2.0, lc, what=(what, M, N, K, split, pads, offs))


@pytest.mark.parametrize("dtype", [pi.F32, pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
def test_ring_of_loose_tiles(gu, oracle, dtype, transA, transB):
    epc = 16 // pi.DTYPE_SIZE[dtype]
    seen = 0
    for vid, name in gu.variants_for(dtype, transA, transB):
        if "_r" not in name:
            continue
        seen += 1
        with gu.pg.Plan(64, 64, 4096, dtype, transA, transB, flags=gu.pg.force_flags(vid)) as p:
            info = dict(w.split("=", 1) for w in p.info().split() if "=" in w)
        bk, stages = int(info["tile"].split("x")[2]), int(info["stages"])
        for tiles, tail, split in [(1, 0, None), (1, 1, None), (stages, 0, None), (stages + 1, bk - 1, None), (2 * stages, epc + 1, 2),
                                   (2 * stages + 1, 0, 3)]:
            _run(gu, oracle, dtype, transA, transB, 64 + epc + 1, 64 + 2 * epc - 1, tiles * bk + tail, vid, split,
                 (tiles % 3, (tiles + 1) % 2), (tail % 3, 1), name)
    assert seen >= 3


@pytest.mark.parametrize("dtype", [pi.F32, pi.BF16])
@pytest.mark.parametrize("transA,transB", [(0, 1), (1, 0)])
def test_leading_dimension_beyond_32_bit_offsets(gu, oracle, dtype, transA, transB):
    vid = next(i for i, n in gu.variants_for(dtype, transA, transB) if "_r64x64" in n)
    ld = 17_000_001                                           # 64 rows of it are over 2^31 bytes in 16 bits, 32 in fp32
    M, N, K = (3, 70, 66) if not transA else (70, 70, 3)
    _run(gu, oracle, dtype, transA, transB, M, N, K, vid, None, (ld - (M if transA else K), 1), (1, 1), "far rows")


@pytest.mark.parametrize("dtype", [pi.F32, pi.F16, pi.BF16])
@pytest.mark.parametrize("transA,transB", list(itertools.product([0, 1], [0, 1])))
def test_no_more_stages_than_k_tiles(gu, oracle, dtype, transA, transB):
    """Fewer K tiles than the ring has stages: a launch's LDS ends with the last of them, the one that K ends in among them."""
    epc = 16 // pi.DTYPE_SIZE[dtype]
    seen = 0
    for vid, name in gu.variants_for(dtype, transA, transB):
        ring = "_m" in name and "q" in name.split("_")[1]
        if not ring and "_r" not in name:
            continue
        seen += 1
        with gu.pg.Plan(64, 64, 4096, dtype, transA, transB, flags=gu.pg.force_flags(vid)) as p:
            info = dict(w.split("=", 1) for w in p.info().split() if "=" in w)
        bm, bn, bk = (int(x) for x in info["tile"].split("x"))
        for tiles in range(1, int(info["stages"]) + 1):
            if ring:                                          # K a whole number of chunks, at and off a tile's end
                _run(gu, oracle, dtype, transA, transB, bm + 2 * epc, 2 * bn, tiles * bk - (tiles % 2) * epc, vid, None, (0, 0), (0, 0), name)
            else:
                _run(gu, oracle, dtype, transA, transB, bm + epc + 1, 2 * bn - 3, tiles * bk - (tiles % 2) * (bk // 2 + 1), vid, None,
                     (tiles % 3, 1), (1, tiles % 2), name)
        _run(gu, oracle, dtype, transA, transB, bm, bn, 3 * bk, vid, 3, (0, 0), (0, 0), name)      # slices of one tile
    assert seen >= 5
