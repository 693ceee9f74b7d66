"""Which kernel the library runs a request on, through its host-only query
gba_fused_plan (no GPU).  The measured choices name their times (MI355X,
microseconds, operands in cache)."""
import ctypes
import random

import pytest

from paper_2006_12645_amd import gba

FAKE = 0x10000  # 16-byte aligned, never dereferenced: the query does not touch memory
LAYOUTS = {"RR": (0, 0), "RC": (0, 1), "CR": (1, 0), "CC": (1, 1)}
MAX_THREADS = (1 << 32) - 1  # of one launch


def desc(M, N, K, layout="RC", pad=0, accum="f32", prologue=False, K2=0, tile=-1, split=0, workspace=0):
    la, lb = LAYOUTS[layout]
    d = gba.new_desc()
    d.layoutA, d.layoutB, d.M, d.N, d.K = la, lb, M, N, K
    d.A, d.lda = FAKE, (K if la == 0 else M) + pad
    d.B, d.ldb = FAKE, (N if lb == 0 else K) + pad
    if K2:
        d.second, d.K2 = gba.GBA_SECOND_ADD, K2
        d.P, d.ldp = FAKE, (K2 if la == 0 else M) + pad
        d.Q, d.ldq = FAKE, (N if lb == 0 else K2) + pad
    d.prologue = gba.GBA_PRO_RELU if prologue else gba.GBA_PRO_NONE
    d.bias_kind, d.bias = gba.GBA_BIAS_ROW, FAKE
    d.act, d.C, d.ldc = gba.GBA_ACT_RELU, FAKE, N
    d.accum = gba.ACCS[accum]
    d.tile_id, d.split_k = tile, split
    if workspace:
        d.workspace, d.workspace_bytes = FAKE, workspace
    return d


def plan(*args, **kw):
    return gba.fused_plan(desc(*args, **kw))


def path(*args, **kw):
    return plan(*args, **kw)["path"]


def test_query():
    assert path(0, 5, 5) == "empty"
    assert plan(4096, 4096, 4096) == {"path": "tile", "bm": 256, "bn": 256, "splits": 1, "threads": 512,
                                      "workgroups": 256}
    assert plan(2048, 2048, 2048) == {"path": "deep", "bm": 128, "bn": 128, "splits": 1, "threads": 512,
                                      "workgroups": 256}
    assert path(4, 4096, 1024) == "few_rows" and path(4095, 4095, 4095) == "unaligned"
    assert path(40, 300, 50, accum="f16") == "general"
    p = plan(64, 512, 32768, workspace=16 << 20)
    assert p["path"] == "tile" and p["splits"] > 1 and p["workgroups"] == 2 * 8 * p["splits"]
    assert plan(64, 512, 32768)["splits"] == 1  # no workspace
    assert gba.lib().gba_fused_plan(ctypes.byref(desc(8, 8, 8)), None) == gba.GBA_EINVAL
    assert gba.lib().gba_fused_plan(ctypes.byref(desc(-1, 8, 8)), ctypes.byref(gba.Plan())) == gba.GBA_EINVAL


@pytest.mark.parametrize("layout,M,N,K", [
    ("RC", 1, 300_000_000, 8),     # 16 columns per 256 threads would be 4.8e9 threads
    ("CC", 16, 140_000_000, 500),  # per 512
    ("RR", 20, 600_000_000, 3), ("CR", 2, 1_000_000_000, 1)])
def test_launch_of_few_rows_stays_in_the_runtimes_limit(layout, M, N, K):
    """A launch has fewer than 2^32 threads; the general kernel, which took
    these requests before the few-row kernel, needs 4 a column."""
    p = plan(M, N, K, layout, pad=1)
    assert p["threads"] * p["workgroups"] <= MAX_THREADS, p


@pytest.mark.parametrize("tile,M,N,split", [(23, 16384, 16384, 64), (21, 32768, 16384, 64), (6, 262144, 65536, 2)])
def test_split_whose_launches_do_not_fit_runs_unsplit(tile, M, N, split):
    """Both launches of a split are checked before the first: tile 23 has 320
    threads per 1024 outputs and split (268M outputs at 64 splits: 5.4e9), the
    second kernel one per four outputs (2^34 of them: 2^32)."""
    p = plan(M, N, 8192, tile=tile, split=split, workspace=1 << 60)
    assert p["splits"] == 1 and p["threads"] * p["workgroups"] <= MAX_THREADS, p


def test_largest_split_that_fits_is_kept():
    assert plan(12288, 16384, 8192, tile=23, split=64, workspace=1 << 60)["splits"] == 64  # 4.03e9 threads


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("M,N,K,pad", [(64, 512, 32767, 1), (64, 512, 32768, 1), (100, 100, 20000, 0), (128, 100, 40001, 0)])
def test_long_reduction_outside_the_fast_path_is_spread_over_the_chip(M, N, K, pad, layout):
    """It cannot be split across workgroups; on the 64x64 tile it would have
    2 to 8 of them."""
    for kw in ({}, {"workspace": 16 << 20}):
        p = plan(M, N, K, layout, pad=pad, **kw)
        assert p["path"] == "few_rows" and p["workgroups"] >= 28, p


def test_requested_split_is_kept_where_the_tile_can_make_it():
    p = plan(64, 512, 1024, split=4, workspace=16 << 20)
    assert p["path"] == "tile" and p["splits"] == 4, p
    for kw in (dict(split=4), dict(split=4, accum="f16", workspace=16 << 20)):
        assert plan(64, 512, 1024, **kw)["splits"] == 1, kw


@pytest.mark.parametrize("layout,M,N,K,want", [("RC", 64, 256, 4096, "few_rows"),   # for a tile of four k-groups
                                               ("RR", 3072, 320, 2496, "deep")])    # for one of two
def test_requested_split_that_no_tile_can_make_changes_nothing(layout, M, N, K, want):
    la, lb = LAYOUTS[layout]
    p = plan(M, N, K, layout, split=4, workspace=1 << 30)
    assert p == plan(M, N, K, layout) and p["path"] == want and p["splits"] == 1, p


@pytest.mark.parametrize("layout,M,N,K,want", [
    # (general, few rows: us)
    ("RC", 9, 47458, 33, "general"),    # 5.2, 17.4
    ("RC", 11, 20121, 486, "general"),  # 8.7, 18.3
    ("RC", 15, 47066, 4393, "general"),  # 87, 113
    ("CC", 24, 25091, 484, "general"),  # 14.1, 29.3
    ("RR", 1, 43509, 48, "general"),    # 6.8, 16.2
    ("RR", 806, 576, 4, "general"),     # 5.3, 8.2
    ("RR", 14, 8449, 4, "general"),     # 5.0, 5.6
    ("RC", 14, 5238, 37, "general"),    # 4.4, 5.2
    ("RC", 22, 8099, 428, "general"),   # 7.7, 8.4
    ("CR", 19, 46576, 292, "general"),  # 25.6, 32.6
    ("RC", 1, 4096, 1024, "few_rows"),  # 10.7, 4.1
    ("RC", 4, 8192, 8192, "few_rows"),  # 96, 22
    ("RC", 22, 5838, 497, "few_rows"),  # 8.0, 6.4
    ("CC", 11, 50184, 928, "few_rows"),  # 80, 43
    ("RR", 8, 13535, 56, "few_rows"),   # 5.8, 5.3
    ("RR", 5, 53525, 457, "few_rows"),  # 41, 26
    ("CR", 20, 40577, 428, "few_rows"),  # 35.2, 36.0
    ("CR", 30, 37922, 474, "few_rows"),  # 47.9, 31.5
])
def test_few_rows_against_the_general_kernel(layout, M, N, K, want):
    assert path(M, N, K, layout, pad=1) == want


def test_few_rows_over_many_columns_of_row_major_b_take_wider_blocks():
    """RR 1 x 43509 x 48: 8.1 us on 16x64 blocks, 16.2 on 16x32."""
    assert plan(5, 53525, 457, "RR", pad=1)["bn"] == 64 and plan(5, 16384, 457, "RR", pad=1)["bn"] == 64
    assert plan(5, 8192, 457, "RR", pad=1)["bn"] == 32


@pytest.mark.parametrize("layout,M,N,K,want", [
    # (tiles, few rows: us)
    ("RC", 256, 256, 1024, "tile"), ("RC", 256, 256, 1152, "few_rows"),  # 4.2, 4.6 at 1024; 9.3, 6.6 at 4096
    ("RR", 656, 624, 1624, "tile"),     # 10.3, 11.3
    ("RR", 64, 1024, 4096, "few_rows"),  # 11.6, 8.2
    ("CR", 872, 576, 2424, "tile"),     # 16.4, 19.7
    ("CR", 224, 1568, 2680, "tile"),    # 16.8, 19.9
    ("CR", 1472, 224, 1696, "tile"),    # 10.2, 12.5
    ("CC", 48, 2048, 2048, "few_rows"),  # 7.8, 6.1
    ("CC", 72, 1536, 1784, "tile"),     # 8.5, 9.8
])
def test_few_rows_against_the_tiles(layout, M, N, K, want):
    assert path(M, N, K, layout) == want


@pytest.mark.parametrize("layout,M,N,K,K2,want", [
    # the same with a second product, for which the tiles start twice
    ("CC", 416, 288, 1856, 512, "few_rows"),  # 8.9, 11.6
    ("RC", 672, 192, 1832, 576, "few_rows"),  # 7.9, 9.7
    ("RR", 512, 384, 1464, 768, "few_rows"),  # 9.9, 11.7
    ("CR", 128, 736, 280, 1536, "few_rows"),  # 8.3, 10.2
    ("CR", 992, 256, 864, 1288, "few_rows"),  # 10.8, 13.3
    ("CR", 416, 1120, 1704, 400, "tile"),     # 19.8, 16.0
    ("CC", 416, 288, 704, 824, "tile"),       # below the least K
])
def test_few_rows_against_the_tiles_with_a_second_product(layout, M, N, K, K2, want):
    assert path(M, N, K, layout, K2=K2) == want


@pytest.mark.parametrize("layout,M,N,K,want", [
    # fp16 accumulation, two workgroups of the four-stage tile per compute
    # unit against the 8-wave tile (us)
    ("RR", 1088, 1792, 3072, 24),  # 31.4, 37.1
    ("RR", 1144, 1120, 1544, 24),  # 17.7, 20.9
    ("RR", 2872, 408, 2240, 24),   # 22.7, 26.7 at K = 2040
    ("RR", 3488, 376, 1352, 20),   # 16.5, 14.0
    ("RR", 2904, 272, 1976, 20),   # 20.0, 17.7
    ("CC", 4032, 320, 4544, 25),   # 37.7, 49.2
    ("CC", 432, 3112, 1216, 19),   # 14.9, 13.7
    ("CC", 1400, 1032, 1656, 25),  # 20.4, 24.7
    ("CC", 512, 4096, 1024, 25),   # 13.4, 16.0
    ("RR", 2048, 1024, 1024, 24),  # 14.2, 17.0
    ("CC", 256, 8192, 2048, 25),   # 21.2, 25.5
    ("RR", 8192, 256, 2048, 24),   # 22.1, 25.3
    ("RR", 512, 4096, 1280, 20),   # 16.6, 13.7
    ("RR", 1024, 2048, 1152, 20),  # 15.6, 13.0
    ("CC", 4096, 512, 1280, 19),   # 14.6, 13.3
    ("RR", 1000, 1000, 512, 24),   # one workgroup per compute unit
])
def test_fp16_four_stage_tile_on_two_rounds(layout, M, N, K, want):
    la, lb = LAYOUTS[layout]
    assert gba.select_tile(M, N, K, la, lb, accum="f16") == want


@pytest.mark.parametrize("layout,M,N,K,want", [
    # fp16 accumulation outside the fast path (us)
    ("CR", 1968, 4802, 1728, 128),  # 166 on 256x256, 77
    ("RC", 3615, 3221, 896, 128),   # 100 on 256x256
    ("RC", 4095, 4095, 4096, 128),
    ("RC", 325, 73, 64, "general"),  # 4.6, 5.4 on 64x64
    ("RC", 1352, 2119, 96, "general"),  # 7.6, 9.2 on 128x128
    ("RR", 325, 73, 64, 64), ("RC", 325, 73, 320, 64),
])
def test_unaligned_fp16(layout, M, N, K, want):
    p = plan(M, N, K, layout, pad=1, accum="f16")
    assert p["path"] == want if want == "general" else (p["path"], p["bm"]) == ("unaligned", want), p


@pytest.mark.parametrize("layout,M,N,K,want", [
    # 256x256, 128x128 (us)
    ("CC", 3081, 3061, 1933, 128),  # 88, 67
    ("CC", 2082, 5583, 1221, 128),  # 63, 51
    ("CC", 4095, 4095, 4095, 256),  # 174, 192
    ("RC", 3081, 3061, 1933, 256),  # 64, 69
    ("RC", 4095, 4095, 4095, 256),  # 142, 195
])
def test_unaligned_256x256_tile(layout, M, N, K, want):
    assert plan(M, N, K, layout, pad=1)["bm"] == want


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("prologue", [False, True])
def test_forcing_the_answered_tile_changes_nothing(layout, prologue):
    """bench.py's mlp_down workload (8192 x 1024 x 4096) forced the id it was
    told and ran the plain 256x128 tile in place of its deep variant."""
    rng, deep = random.Random(5), 0
    shapes = [(8192, 1024, 4096), (2048, 2048, 2048), (1024, 1920, 1280)] + [
        tuple(8 * rng.randint(4, 512) for _ in range(3)) for _ in range(400)]
    for M, N, K in shapes:
        want = plan(M, N, K, layout, prologue=prologue)
        if want["path"] not in ("tile", "deep"):
            continue
        deep += want["path"] == "deep"
        t = gba.fused_tile(desc(M, N, K, layout, prologue=prologue))
        assert plan(M, N, K, layout, prologue=prologue, tile=t) == want, (M, N, K)
    assert deep >= 10
    p = plan(2048, 2048, 2048, layout, tile=4, split=2, workspace=1 << 30)
    assert p["path"] == "tile" and p["splits"] == 2  # a split is kept


def test_leading_dimensions_beyond_32_bit_offsets_take_the_general_kernel():
    for M, want in ((5, "few_rows"), (70, "unaligned")):
        for layout in LAYOUTS:
            for over in (0, 1):
                d = desc(M, 75, 130, layout)
                d.lda = d.ldb = (1 << 23) - 1 + over
                assert gba.fused_plan(d)["path"] == ("general" if over else want)
