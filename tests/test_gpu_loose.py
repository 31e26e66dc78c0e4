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
@pytest.mark.parametrize("operand", ["A", "B"])
@pytest.mark.parametrize("along_k", [True, False])
@pytest.mark.parametrize("beyond", [False, True])
def test_leading_dimension_at_the_limit_of_the_copies(gu, oracle, dtype, operand, along_k, beyond):
    """A 64x64 tile with a whole K tile and a tail; its last row (along K) or k-row ends just within 2^31 bytes of its first, by direct
    copies, or beyond them, where 32-bit offsets would overflow, through registers."""
    import torch
    es = pi.DTYPE_SIZE[dtype]
    bk = 128 // es
    strides = 64 if along_k else bk                           # rows of the tile that lie one leading dimension apart
    ld = (2 ** 31 + 2 ** 23) // ((strides - 1) * es) | 1 if beyond else 2 ** 31 // (strides * es) - 129 - 128 * (not along_k)
    assert ((strides - 1) * ld * es > 2 ** 31) == beyond
    M, N, K = 64 + 5, 64 + 7, bk + 3
    transA, transB = (int(not along_k), 1) if operand == "A" else (0, int(along_k))
    vid = next(i for i, n in gu.variants_for(dtype, transA, transB) if "_r64x64" in n)
    la, lb = (pi.logical_matrix(61, i, *s, "uniform", 1.0, dtype) for i, s in enumerate(((M, K), (K, N))))
    A, B = pi.store(la, bool(transA)), pi.store(lb, bool(transB))
    far = A if operand == "A" else B
    rows, cols = far.shape
    buf = torch.full((1 + (rows - 1) * ld + cols,), float("nan"), dtype=torch.float32 if es == 4 else torch.bfloat16, device="cuda")
    torch.as_strided(buf, (rows, cols), (ld, 1), 1).copy_(gu.to_dev(far).view(buf.dtype))
    dA, dB = (buf if m is far else gu.to_dev(m) for m in (A, B))
    dC = gu.to_dev(gu.nan_fill(M, N, dtype))
    lda, ldb = (ld if m is far else m.shape[1] for m in (A, B))
    off = [es if m is far else 0 for m in (A, B)]
    print(operand, along_k, M, N, K, lda, ldb, flush=True)
    with gu.pg.Plan(M, N, K, dtype, transA, transB, lda, ldb, N, gu.pg.force_flags(vid, 1)) as plan:
        plan.run(1.0, dA.data_ptr() + off[0], dB.data_ptr() + off[1], 0.0, dC.data_ptr(), 0, 0, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    got = pi.to_f64(np.ascontiguousarray(gu.from_dev(dC, dtype)), dtype)
    gu.check_against_oracle(oracle, got, dtype, transA, transB, M, N, K, 1.0, A, B, 0.0, None, what=(operand, along_k, ld))


@pytest.mark.parametrize("dtype", [pi.F32, pi.BF16])
@pytest.mark.parametrize("transA,transB", [(0, 1), (1, 0)])
def test_few_rows_far_apart(gu, oracle, dtype, transA, transB):
    """Three rows of A, or three k, a leading dimension apart that is too large for 64 of them."""
    vid = next(i for i, n in gu.variants_for(dtype, transA, transB) if "_r64x64" in n)
    ld = 17_000_001
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
