"""Which route a plan takes: aligned copies, any-alignment kernels, ring kernels (no GPU needed)."""
import itertools
import os
import subprocess
import sys

import pytest

import paper_2512_19018_amd as pg

SHIPPED_TABLE = os.path.join(os.path.dirname(pg.__file__), "peak_gemm_tuning.txt")
DTYPES = {"f32": (pg.PEAK_DT_F32, 4), "f16": (pg.PEAK_DT_F16, 2), "bf16": (pg.PEAK_DT_BF16, 2)}


def plan(dt, ta, tb, M, N, K, pad=(0, 0, 0), flags=0):
    p = pg.Plan(M, N, K, DTYPES[dt][0], ta, tb, (M if ta else K) + pad[0], (K if tb else N) + pad[1], N + pad[2],
                flags=flags)
    info = p.info()
    fields = dict(w.split("=", 1) for w in info.split() if "=" in w)
    return p, fields["variant"].split(":")[1], int(fields["split"]), int(fields["pack"]), fields["unaligned"]


@pytest.mark.parametrize("dt,ta,tb", list(itertools.product(DTYPES, (0, 1), (0, 1))))
def test_every_form_takes_a_kernel_that_can_read_it(dt, ta, tb):
    """Rows that do not fill 16-byte chunks go to a kernel for any alignment or through copies of just those operands."""
    chunk = 16 // DTYPES[dt][1]
    for M, N, K, pa, pb in itertools.product((100, 1024, 2049), (96, 1000, 2051), (512, 1031), (0, 1, chunk), (0, 1, chunk)):
        p, name, _, pack, alt = plan(dt, ta, tb, M, N, K, (pa, pb, 0))
        tail = K % chunk != 0
        odd_a = tail or ((M if ta else K) + pa) % chunk != 0 or (ta and M % chunk != 0)
        odd_b = tail or ((K if tb else N) + pb) % chunk != 0 or (not tb and N % chunk != 0)
        any_alignment = name.startswith(dt + "_r") or "skinny" in name
        if pack:
            assert M > 64 and pack == (1 if odd_a else 0) | (2 if odd_b else 0)
            rows = (pack & 1) * M * K + (pack >> 1) * N * K
            assert p.workspace_bytes >= rows * DTYPES[dt][1]
            assert not any_alignment and alt.startswith(dt + "_r")
        elif odd_a or odd_b:
            # (the "_d..._nn" kernels mask the columns of B themselves; with K along no row the direct copies end with K)
            masked = name.endswith("_nn") and "_d" in name and not odd_a and (N + pb) % chunk == 0
            rows_of_k = ta and not tb and (M + pa) % chunk == M % chunk == 0 and (N + pb) % chunk == N % chunk == 0
            assert any_alignment or masked or rows_of_k, (M, N, K, pa, pb, name)
        # whatever the operands' addresses, a kernel without alignment conditions stands by
        assert any_alignment or alt.startswith(dt + "_r"), (name, alt)


@pytest.mark.parametrize("dt", DTYPES)
def test_partials_of_ring_and_any_alignment_kernels_fit_the_fixed_array(dt):
    for M, N, K, odd in itertools.product((33, 100, 700, 1700), (40, 512, 3072, 8192), (256, 3000, 16384), (0, 1)):
        p, name, split, pack, _ = plan(dt, 0, 1, M, N, K, (odd, odd, 0))
        if not pack and (name.startswith(dt + "_r") or "q" in name):
            assert split * M * N * 4 <= pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES or split == 1
            assert p.workspace_bytes <= pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES


@pytest.mark.parametrize("dt,ta,tb,M,N,K,ring", [
    ("f32", 0, 1, 504, 1396, 2380, True),        # the large tile only with a K split
    ("f32", 0, 0, 112, 208, 816, True),
    ("f32", 1, 1, 2560, 1340, 2164, False),      # the large tile unsplit
    ("f32", 0, 0, 2048, 4096, 32, False),        # K too short for many rounds of small tiles
    ("bf16", 0, 0, 4096, 4096, 64, False),
    ("bf16", 0, 1, 100, 4096, 4096, True),
    ("f16", 0, 1, 64, 4096, 8192, True),         # 33 to 64 rows against a small streamed operand
    ("f16", 0, 1, 32, 4096, 8192, False),
    ("bf16", 0, 1, 50, 23232, 1152, False),      # ... but not where the streaming kernel needs no K split
    ("bf16", 0, 1, 50, 6144, 4992, False),       # nor where a slice of the ring kernel is deep
    ("bf16", 0, 1, 40, 4800, 7552, True),
    ("bf16", 0, 1, 64, 8192, 2688, True),
    ("f16", 0, 0, 64, 6848, 4160, True),
    ("f16", 0, 1, 48, 13888, 1152, True),        # unsplit in 64-column tiles: level cold, ring ahead warm
    ("bf16", 0, 0, 64, 384, 256, True),          # ... or because K is too short for slices
    ("bf16", 0, 1, 64, 1728, 768, True),
    ("bf16", 0, 1, 59, 33088, 768, True),        # unsplit in more than a round
    ("f16", 0, 1, 36, 11008, 2304, True),        # the streaming kernel's slices spill into a second round
    ("bf16", 0, 1, 62, 5632, 6272, False),
    ("bf16", 0, 0, 46, 18368, 2048, False),      # B stored K x N: a second round of ring tiles on a long K
    ("f16", 0, 0, 37, 10112, 3200, True),        # ring tiles, not the 64x128 ones
    ("bf16", 0, 0, 43, 26432, 1408, True),
    ("bf16", 1, 0, 40, 12800, 1024, True),       # A stored K x M: no transposition first
    ("f16", 1, 1, 56, 24128, 1536, True),
    ("f16", 1, 0, 32, 4096, 8192, False),
    ("bf16", 1, 1, 64, 8192, 8192, False),       # too large an operand to be read by small tiles
    ("bf16", 1, 1, 33, 8192, 2048, False),       # rows of A that the ring kernels cannot copy
    ("bf16", 0, 1, 8192, 8192, 8192, False),
])
def test_ring_kernels_where_they_pay(dt, ta, tb, M, N, K, ring):
    _, name, _, _, _ = plan(dt, ta, tb, M, N, K)
    assert ("q" in name.split("_")[1]) == ring, name


# 64 rows, unsplit with 64 columns per tile against 128 and a K split (bf16, us, the operand cold in the caches):
# 16384x8192 50.1 / 56.9, 13312x4096 26.1 / 27.4, 13504x8320 44.2 / 49.9, 14080x12928 80.0 / 77.9, 13312x10624 62.4 / 57.9, 16320x13952 87.5 / 90.2,
# 16384x15488 103 / 97
@pytest.mark.parametrize("N,K,columns", [(13312, 4096, 64), (13504, 8320, 64), (13312, 10624, 128), (14080, 12928, 128), (16384, 8192, 64),
                                         (16320, 13952, 64), (16384, 15488, 128), (16448, 14080, 128), (25664, 14080, 128),
                                         (26624, 14080, 128)])
def test_streaming_tiles_of_64_columns_only_in_one_round(N, K, columns):
    _, name, _, _, _ = plan("bf16", 0, 1, 64, N, K)
    assert name == "bf16_skinny_m64n%dk128s3_nt" % columns


@pytest.mark.parametrize("row,sizes", [
    ("bf16 0 1 4095 4095 4095 bf16_r128x128_nt 1", (4095, 4095, 4095)),
    ("bf16 0 1 1023 2047 3001 bf16_r128x64_nt 4", (1023, 2047, 3001)),
    ("f32 1 0 2049 3001 1023 f32_r64x64_tn 1", (2049, 3001, 1023)),
])
def test_table_rows_of_unaligned_products_are_the_plan(tmp_path, row, sizes):
    """Variant and split of the row, without copies that the row does not name; other shapes still get them."""
    dt, ta, tb, _, _, _, variant, split = row.split()
    args = (dt, int(ta), int(tb))
    assert plan(*args, *sizes)[3] == 3                           # the cost model's choice: aligned copies of both operands
    table = tmp_path / "table.txt"
    table.write_text(row + "\n")
    try:
        assert pg.peak_gemm_load_tuning(str(table)) == 1
        p, name, s, pack, _ = plan(*args, *sizes)
        assert (name, s, pack) == (variant, int(split), 0)
        assert p.workspace_bytes == (s * sizes[0] * sizes[1] * 4 if s > 1 else 0)
        M, N, K = sizes
        assert plan(*args, M + 2, N, K)[3] == 3
    finally:
        pg.peak_gemm_load_tuning(SHIPPED_TABLE)


def test_tuner_leaves_plans_that_no_row_can_ask_for():
    """A row is taken as it is: one for a product whose own plan makes aligned copies or cuts its last round would lose that."""
    from paper_2512_19018_amd import tune
    assert tune.beyond_rows(plan("bf16", 0, 1, 4095, 4095, 4095)[0].info()) == "aligned copies"
    assert tune.beyond_rows(plan("bf16", 0, 1, 4096, 5120, 5120, flags=pg.force_flags(streamk=True))[0].info()) == "stream-K"
    assert tune.beyond_rows(plan("bf16", 0, 1, 8192, 8192, 8192)[0].info()) is None
    assert tune.beyond_rows(plan("bf16", 0, 1, 101, 103, 107)[0].info()) is None


# (as many slices as fill the chip once, rounded up, were 2, 5, 3 and 3: a second round with few workgroups in it)
@pytest.mark.parametrize("dt,ta,tb,M,N,K,splits", [("f16", 0, 1, 16, 8960, 7680, 3), ("f32", 1, 0, 37, 6592, 16128, 9),
                                                   ("f32", 0, 0, 35, 11840, 2560, 5), ("bf16", 0, 0, 30, 23296, 9344, 2)])
def test_streaming_slices_do_not_spill_into_a_thin_round(dt, ta, tb, M, N, K, splits):
    _, name, split, _, _ = plan(dt, ta, tb, M, N, K)
    assert "skinny" in name and split == splits


@pytest.mark.parametrize("dt,ta,tb", list(itertools.product(DTYPES, (0, 1), (0, 1))))
def test_streaming_slices_and_copy_fit_the_fixed_array(dt, ta, tb):
    """... unless already the slices that fill the chip once ask for more, which only a K beyond 100000 does."""
    streaming = beyond = 0
    for M, N, K in itertools.product((1, 16, 17, 32, 33, 48, 64), (2048, 8960, 13312, 28672, 40960), (2048, 7680, 16384, 28672, 131072)):
        p, name, split, _, _ = plan(dt, ta, tb, M, N, K)
        if "skinny" not in name:
            continue
        streaming += 1
        if p.workspace_bytes > pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES:
            columns = int(p.info().split("tile=")[1].split()[0].split("x")[1])
            tiles = -(-N // columns)
            assert K == 131072 and split == max(1, (256 + tiles // 4) // tiles), (M, N, K, split)
            beyond += 1
    assert streaming > 100 and beyond < 20


def test_streaming_slices_fill_the_compute_units_there_are():
    code = ("import paper_2512_19018_amd as pg\n"
            "for N in (2048, 4096, 8192):\n"
            "    print(pg.Plan(16, N, 16384, pg.PEAK_DT_BF16, 0, 1).info().split('grid=')[1].split()[0])")
    for cu in (64, 128, 256):
        env = dict(os.environ, PEAK_GEMM_NUM_CU=str(cu), PYTHONPATH=os.path.dirname(os.path.dirname(pg.__file__)))
        out = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, check=True).stdout.split()
        assert all(cu * 3 // 4 <= int(g) <= cu * 5 // 4 for g in out), (cu, out)


@pytest.mark.parametrize("dt", ("f16", "bf16"))
@pytest.mark.parametrize("tb,M,N,K,stages", [(0, 192, 2816, 1088, 3), (1, 195, 3088, 472, 3), (0, 192, 2816, 28 * 64, 3), (0, 192, 2816, 29 * 64, 5),
                                             (0, 320, 2688, 20 * 64, 3), (0, 320, 2688, 21 * 64, 5), (1, 1024, 1024, 4480, 5)])
def test_ring_stages_by_the_depth_of_a_slice(dt, tb, M, N, K, stages):
    _, name, split, _, _ = plan(dt, 0, tb, M, N, K)
    assert "_m64x64q%d_" % stages in name and split == 1


# B stored K x N in whole-chunk rows with an N of no whole chunks: the ring kernels cannot read it, the large tiles that mask the edge can
PADDED_B = [("f32", 112, 109, 72), ("f32", 614, 359, 84), ("f32", 384, 105, 5844), ("bf16", 512, 1001, 1024), ("f16", 1328, 204, 384),
            ("f16", 272, 2514, 416), ("bf16", 1753, 157, 544), ("f32", 524, 3826, 3752), ("f32", 345, 5647, 4848), ("f32", 324, 5531, 3416)]


@pytest.mark.parametrize("dt,M,N,K", PADDED_B)
def test_masked_large_tiles_stand_against_the_kernels_for_any_alignment(dt, M, N, K):
    chunk = 16 // DTYPES[dt][1]
    p, name, split, pack, _ = plan(dt, 0, 0, M, N, K, (0, -N % chunk, 0))
    assert name.startswith(dt + "_r") and not pack, (name, pack)
    assert p.workspace_bytes <= pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES


def test_partials_with_a_padded_b_fit_the_fixed_array():
    """fp32, where the masked tiles' own split would ask for more: peak_gemm_run_static takes every one."""
    for M, N, K in itertools.product((345, 524, 858, 1060), (1509, 2809, 3183, 3826, 5647), (1032, 3264, 4848, 6336)):
        p, name, _, pack, _ = plan("f32", 0, 0, M, N, K, (0, -N % 4, 0))
        if not pack:
            assert p.workspace_bytes <= pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES, (M, N, K, name)
        assert pg.peak_gemm_run_static(p.handle, 1.0, 0, 0, 0.0, 0, 0) != pg.PEAK_ERR_WORKSPACE, (M, N, K, name)


# (256x128 tiles, which a ring that keeps all its stages however few K tiles there are was priced against, took 6.7 to 8.2 us, these 5.8 to 7.6)
@pytest.mark.parametrize("dt,ta,tb,M,N,K", [("bf16", 1, 1, 3144, 1744, 64), ("f16", 0, 1, 1088, 4552, 64), ("bf16", 0, 0, 1696, 3416, 64),
                                            ("bf16", 0, 0, 672, 5960, 64), ("f16", 1, 0, 2048, 2944, 64), ("f16", 0, 0, 1024, 5392, 128),
                                            ("f16", 1, 0, 3080, 1576, 128), ("f16", 1, 1, 2552, 3096, 64), ("bf16", 0, 0, 6248, 680, 64)])
def test_few_k_tiles_go_to_ring_tiles(dt, ta, tb, M, N, K):
    _, name, split, _, _ = plan(dt, ta, tb, M, N, K)
    assert "q" in name.split("_")[1] and split == 1, name


# us with the price per round of workgroups, then these: 5.9, 5.3; 7.5, 6.7; 5.8, 5.3; 5.75, 5.2; 5.9, 5.3; 12.5, 10.5; 12.6, 10.6
@pytest.mark.parametrize("dt,ta,tb,M,N,K,variant", [
    ("f32", 1, 0, 449, 1527, 55, "f32_r64x64_tn"), ("f32", 0, 0, 2371, 297, 105, "f32_r64x64_nn"), ("f32", 0, 0, 83, 5877, 57, "f32_r64x64_nn"),
    ("f32", 1, 0, 335, 2013, 41, "f32_r64x64_tn"), ("f32", 1, 0, 8117, 87, 59, "f32_r64x64_tn"),
    ("bf16", 1, 0, 1616, 4864, 144, "bf16_m128x64q3_tn"), ("f16", 1, 0, 1120, 6576, 176, "f16_m128x64q3_tn")])
def test_tiles_of_a_short_k(dt, ta, tb, M, N, K, variant):
    assert plan(dt, ta, tb, M, N, K)[1] == variant


def test_copies_by_price_without_steps_in_k():
    """Blocks of 1023 x 2047: copies from one K on, wherever rows of the larger matrices end."""
    packed = [plan("bf16", 0, 1, 1023, 2047, K, (6, 6, 6))[3] == 3 for K in range(515, 4100, 24)]
    assert packed == sorted(packed) and not packed[0] and packed[-1]
    for K in (999, 1001, 2999, 3001):
        assert plan("bf16", 0, 1, 1023, 2047, K, (6, 6, 6))[3] == plan("bf16", 0, 1, 1023, 2047, K + 2, (6, 6, 6))[3]


def test_copies_of_even_leading_dimensions_wait_for_the_base():
    """16 bits: 2050x2042x1026 takes 24 us without copies where both bases are even, 37 where they are odd, and 29 with copies."""
    for dt, M, N, K, pad, odd in (("bf16", 2050, 2042, 1026, 0, 1), ("f16", 2049, 2047, 1031, 1, 1), ("bf16", 2049, 2047, 1031, 0, 0),
                                  ("bf16", 4096, 4096, 4095, 1, 0)):
        p = plan(dt, 0, 1, M, N, K, (pad, pad, 0))[0]
        assert "pack=3 oddbase=%d " % odd in p.info(), p.info()


# us with copies and without: 28 and 32, 70 and 109; 37 and 30, 116 and 94, 114 and 102, 94 and 78, 72 and 59
@pytest.mark.parametrize("dt,ta,tb,M,N,K,copies", [
    ("bf16", 0, 1, 563, 5571, 1817, True), ("f16", 0, 1, 1647, 8173, 2121, True), ("f32", 1, 0, 797, 2311, 673, False),
    ("f32", 1, 0, 685, 2997, 2121, False), ("f32", 1, 1, 1753, 3463, 907, False), ("f32", 1, 0, 629, 2419, 2833, False),
    ("f32", 1, 0, 1547, 843, 2115, False)])
def test_copies_where_they_pay(dt, ta, tb, M, N, K, copies):
    assert (plan(dt, ta, tb, M, N, K)[3] != 0) == copies


def test_partials_beyond_the_fixed_array_stand_against_the_kernels_for_any_alignment():
    """fp32: ten slices of 256x256 tiles ask for 43 MB, the kernels for any alignment are 20 % ahead by price and within the array."""
    p, name, _, _, _ = plan("f32", 0, 1, 192, 5908, 7808, (0, 8, 0))
    assert name.startswith("f32_r") and p.workspace_bytes <= pg.PEAK_GEMM_STATIC_WORKSPACE_BYTES


# relative error of one sum for all k in ring tiles, then of these: 1.6e-6, 3.5e-7; 6.4e-7, 2.7e-7; 1.2e-6, 2.8e-7; 7.9e-7, 3.3e-7; 7.1e-7, 3.6e-7
@pytest.mark.parametrize("ta,tb,M,N,K", [(0, 1, 192, 4304, 7576), (0, 1, 3336, 168, 4976), (1, 0, 4120, 192, 4464), (1, 1, 172, 3592, 7824),
                                         (1, 1, 5912, 168, 6364)])
def test_deep_fp32_products_in_tiles_of_several_sums(ta, tb, M, N, K):
    _, name, split, _, _ = plan("f32", ta, tb, M, N, K)
    assert name.startswith("f32_r64x") and split >= 3


# one sum per element in 128x128, four in 64x64: a result of K in the hundreds is off by 3.6e-7 and 2.6e-7
@pytest.mark.parametrize("ta,tb,M,N,K", [(1, 1, 6204, 3846, 393), (1, 1, 979, 3200, 68), (0, 1, 2809, 3841, 1255), (1, 0, 1043, 2179, 2697)])
def test_fp32_tiles_of_one_sum_only_far_ahead(ta, tb, M, N, K):
    assert "_r128x128" not in plan("f32", ta, tb, M, N, K, (1, 1, 0))[1]


# 64x32 tiles in place of 64x64 with one or two K tiles: a third workgroup per CU to start (748x1752x32 NN 5.11 us and 4.76)
@pytest.mark.parametrize("ta,tb,M,N,K", [(0, 0, 748, 1752, 32), (1, 0, 2348, 492, 12), (0, 1, 240, 4740, 16), (0, 1, 968, 1268, 64)])
def test_fp32_64x64_rings_at_short_k(ta, tb, M, N, K):
    assert "_m64x64q3" in plan("f32", ta, tb, M, N, K)[1]


@pytest.mark.parametrize("dt,ta,tb,M,N,K", [
    ("bf16", 0, 1, 1024, 5120, 5120), ("f16", 0, 0, 2048, 4096, 14336), ("bf16", 0, 0, 2048, 28672, 8192), ("bf16", 1, 0, 2048, 28672, 8192),
    ("bf16", 1, 1, 2048, 28672, 8192), ("bf16", 0, 1, 1024, 4096, 14336), ("bf16", 0, 1, 2048, 2048, 512), ("f32", 0, 0, 3072, 3072, 3072)])
def test_layer_shapes_run_without_a_workspace(dt, ta, tb, M, N, K):
    """Products of layers that peak_gemm_run_static, and a run without workspace, have always taken."""
    p, name, split, _, _ = plan(dt, ta, tb, M, N, K)
    small = dict(w.split("=", 1) for w in p.info().split() if "=" in w)["small"]
    assert p.workspace_bytes == 0 or small != "none", p.info()
