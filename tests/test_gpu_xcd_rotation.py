"""K walked from another tile on each XCD: K tiles a multiple of eight or not, one that K ends in, slices."""
import numpy as np
import pytest

import peak_inputs as pi

pytestmark = pytest.mark.gpu

TILES = ["m256x256w4a3", "m256x128w4a3", "m128x128w4a3", "m128x128w4a5", "m128x128k128w4a3", "m128x64q3", "m64x64q3", "m64x64q5"]


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
    _exact(gu, oracle, "%s_%s_%s" % (pi.DTYPE_NAMES[dtype], tile, "tt" if transA else "nt"), dtype, transA, K, split)


# two waves along K, A along K only
@pytest.mark.parametrize("dtype", [pi.BF16, pi.F16])
@pytest.mark.parametrize("K,split", [(4096, 1), (4168, 1), (8856, 2)])
def test_with_waves_that_share_k(gu, oracle, dtype, K, split):
    _exact(gu, oracle, "%s_m32x64k128q3_nt" % pi.DTYPE_NAMES[dtype], dtype, 0, K, split)


def _exact(gu, oracle, name, dtype, transA, K, split):
    pg = gu.pg
    M, N = 264, 1096                                        # workgroups on every XCD
    vid = _variant(gu, name)
    A, B = _ints(dtype, transA, 1, M, N, K, 8400)
    rows = [0, 1, 127, 128, 255, 256, 263]
    ref = oracle.gemm(dtype, transA, 1, M, N, K, 1.0, A, B, 0.0, None, rows=rows)
    got, _, info = gu.run_gemm(dtype, transA, 1, M, N, K, 1.0, 0.0, A, B, gu.nan_fill(M, N, pi.F32), flags=pg.force_flags(variant=vid, split=split), cdtype=pi.F32)
    assert (" xcdrot=%d " % (split == 1 or "256x256" not in name)) in info, info          # (slices of the largest tile start together)
    assert np.array_equal(got[rows], ref), info             # small integers: exact in fp32 in any order


# equal rows of A: one order of the sum in every tile without the rotation, another on each XCD with it
@pytest.mark.parametrize("name", ["bf16_m128x128w4a3_nt", "bf16_m64x64q5_nt", "f16_m256x256w4a3_nt"])
def test_the_rotation_is_seen_in_the_last_bits(gu, oracle, name, monkeypatch):
    pg = gu.pg
    dtype = pi.BF16 if name.startswith("bf16") else pi.F16
    M, N, K = 1024, 1152, 8192                              # columns of tiles that lie on more than one XCD
    g = np.random.default_rng(46)
    import torch
    bits = lambda x: torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16 if dtype == pi.BF16 else torch.float16).view(torch.int16).numpy().view(np.uint16)
    A, B = bits(np.repeat(g.uniform(-1, 1, (1, K)), M, 0)), bits(g.uniform(-1, 1, (N, K)))
    ref, bound = gu.elementwise_bound(oracle, dtype, 0, 1, M, N, K, 1.0, A, B, 0.0, None, [0], cdtype=pi.F32)
    flags = pg.force_flags(variant=_variant(gu, name), split=1)
    for on in (True, False):
        if not on:
            monkeypatch.setenv("PEAK_GEMM_ROT", "0,0")
        got, _, info = gu.run_gemm(dtype, 0, 1, M, N, K, 1.0, 0.0, A, B, gu.nan_fill(M, N, pi.F32), flags=flags, cdtype=pi.F32)
        assert (" xcdrot=%d " % on) in info, info
        gu.assert_elementwise(got, np.repeat(ref, M, 0), np.repeat(bound, M, 0), info)
        assert bool((got == got[:1]).all()) != on, info
