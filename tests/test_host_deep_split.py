"""Few tiles and a deep K in 16 bits: the 256x256 tile in slices that fill the chip, with the plan of fewer partials behind it."""
import itertools

import pytest

import paper_2512_19018_amd as pg

DTYPES = {"f16": pg.PEAK_DT_F16, "bf16": pg.PEAK_DT_BF16}


def fields_of(dt, ta, tb, M, N, K, pad=0, flags=0):
    with pg.Plan(M, N, K, dt, ta, tb, (M if ta else K) + pad, (K if tb else N) + pad, N, flags=flags) as p:
        return dict(w.split("=", 1) for w in p.info().split() if "=" in w), p.workspace_bytes


@pytest.mark.parametrize("dt,ta,tb", list(itertools.product(DTYPES, (0, 1), (0, 1))))
@pytest.mark.parametrize("M,N,K,deep", [
    (392, 5504, 11392, True), (648, 2560, 24768, True),
    (392, 5504, 7000, False),         # operands that the last-level cache holds
    (392, 5504, 2048, False),         # a slice too short
    (4096, 4096, 14336, False),       # tiles enough without slices
    (64, 8192, 16384, False)])        # streamed
def test_when_the_slices_are_taken(dt, ta, tb, M, N, K, deep):
    f, nbytes = fields_of(DTYPES[dt], ta, tb, M, N, K)
    assert (f["small"] != "none") == deep, f
    if deep:
        split, ktiles = int(f["split"]), int(f["ktiles/slice"])
        tiles = -(-M // 256) * -(-N // 256)
        assert ":%s_m256x256w4a3_" % dt in f["variant"] and f["small"].startswith(dt + "_m")
        assert split > 1 and tiles * split <= 256 and ktiles * split >= -(-K // 64) and ktiles >= 12
        assert 4 * split * M * N <= 96e6 and nbytes >= 4 * split * M * N


@pytest.mark.parametrize("dt,ta,tb,M,N,K,deep", [
    # operands that fit the last-level cache; slices over the plan of fewer partials, from there and from HBM:
    ("f16", 1, 1, 320, 7168, 7168, False), ("f16", 1, 1, 384, 6643, 9088, False),          # 0.83 and 1.06, 0.84 and 1.09
    ("f16", 0, 0, 271, 2304, 18800, False), ("f16", 0, 0, 4384, 352, 11840, False),        # 0.87 and 1.15, 0.86 and 1.12
    ("bf16", 0, 0, 391, 5504, 11392, True), ("bf16", 0, 0, 512, 4096, 14336, True),        # 1.10 and 1.52, 0.96 to 0.98 and 1.22
    ("bf16", 1, 0, 640, 4160, 11072, True),                                                # 1.02 and 1.47
    # ... and that do not
    ("bf16", 0, 0, 144, 4992, 27752, True), ("f16", 0, 0, 5376, 384, 24896, True)])        # 1.37, 1.11
def test_products_that_a_program_may_repeat_with_operands_in_the_cache(dt, ta, tb, M, N, K, deep):
    f, _ = fields_of(DTYPES[dt], ta, tb, M, N, K)
    assert (f["small"] != "none") == deep, f


def test_only_the_selectors_own_choice_changes():
    M, N, K = 392, 5504, 11392
    own, _ = fields_of(pg.PEAK_DT_BF16, 0, 0, M, N, K)
    f, _ = fields_of(pg.PEAK_DT_BF16, 0, 0, M, N, K, flags=pg.force_flags(split=2))
    assert f["small"] == "none", f
    assert own["small"] != "none"
    # an ordinary K split: neither what rules hybrid stream-K out nor what asks for it, without a last round to cut, changes it
    for streamk in (False, True):
        f, _ = fields_of(pg.PEAK_DT_BF16, 0, 0, M, N, K, flags=pg.force_flags(streamk=streamk))
        assert f == own, (streamk, f)
    f, _ = fields_of(pg.PEAK_DT_BF16, 0, 0, M, N, K, pad=1)       # no rows for the 256x256 tile's copies
    assert f["small"] == "none"
    f, _ = fields_of(pg.PEAK_DT_F32, 0, 0, M, N, K)
    assert f["small"] == "none"
