"""CPU checks of the rules that choose a kernel and its grid by size, through the library's host-only plan queries: launch
limits (what one kernel's grid can hold must not fail because the rule takes another) and the choices themselves."""

import ctypes
import os

import pytest

from paper_2606_20381_amd import ufp4 as U

DENSE, RAGGED_M, RAGGED_K = 0, 1, 2


@pytest.fixture(scope="module")
def plan():
    if not os.path.exists(U.library_path()):
        pytest.skip("libufp4.so not built")
    return ctypes.CDLL(U.library_path())


def mx_kernel(plan, mode, m, n, red, groups=1, a_rows=None):
    """(tile, threads of the grid in x) of a power-of-two-scale GEMM; A rows of a ragged-M problem: every group padded."""
    t = ctypes.c_int64()
    if a_rows is None:
        a_rows = (m + 127 * groups) // 128 * 128 if mode == RAGGED_M else m
    k = plan.ufp4_plan_gemm_mx(mode, *map(ctypes.c_int64, (m, n, red)), ctypes.c_int32(groups), ctypes.c_int64(a_rows),
                               ctypes.byref(t))
    return (256, 128, 64)[k], t.value


KERNELS = ("128x128", "128x128 in two K groups", "128x64", "32x32", "64x64")


def gemm_kernel(plan, mode, fmt, m, n, red, groups=1):
    return plan.ufp4_plan_gemm(mode, fmt, *map(ctypes.c_int64, (m, n, red)), ctypes.c_int32(groups))


# us of each of KERNELS
RAGGED_M_TIMES = [  # format, tokens, columns, reduction, groups
    (U.UNIFORM, 1273, 5248, 256, 128, (122.0, 209.9, 132.6, 165.1, 124.3)),
    (U.UNIFORM, 600, 1536, 256, 256, (66.2, 121.3, 78.8, 96.1, 71.3)),
    (U.UNIFORM, 3124, 1280, 1152, 1, (34.8, 44.2, 31.7, 38.8, 28.1)),
    (U.UNIFORM, 9827, 384, 1024, 16, (34.4, 42.7, 30.4, 40.3, 27.0)),
    (U.UNIFORM, 6652, 640, 384, 32, (17.7, 24.3, 21.3, 32.2, 20.8)),
    (U.UNIFORM, 2098, 2304, 1536, 8, (46.5, 55.0, 57.0, 59.4, 46.0)),
    (U.E2M1, 10780, 256, 384, 32, (12.7, 13.5, 12.6, 22.1, 16.4)),
    (U.E2M1, 725, 1152, 256, 128, (29.0, 45.3, 39.7, 35.2, 29.3)),
    (U.E2M1, 18189, 3712, 512, 64, (209.0, 316.9, 281.9, 481.7, 266.6)),
]


def _assert_no_slower_than_the_large_tile(plan, mode, fmt, m, n, red, groups, us):
    """The kernel taken is within 4% of the 128 x 128 one (the spread that the rule grants it) or faster."""
    k = gemm_kernel(plan, mode, fmt, m, n, red, groups)
    assert us[k] <= 1.04 * us[0], KERNELS[k]


SHORT_TIMES = [  # mode, format, rows, columns, reduction: few blocks, more than three 32 x 32 workgroups per CU
    (DENSE, U.UNIFORM, 240, 5328, 160, (7.3, 8.4, 5.7, 8.3, 7.0)),
    (DENSE, U.UNIFORM, 96, 12192, 128, (6.9, 7.9, 5.3, 7.3, 6.4)),
    (DENSE, U.E2M1, 128, 11056, 192, (7.4, 8.1, 6.2, 8.4, 7.2)),
    (DENSE, U.E2M1, 3488, 416, 128, (6.7, 8.2, 5.5, 8.0, 6.2)),
    (RAGGED_K, U.UNIFORM, 512, 2688, 112, (7.0, 7.8, 5.9, 9.6, 7.0)),
    (RAGGED_K, U.E2M1, 1792, 768, 128, (7.4, 8.7, 6.3, 9.7, 7.1)),
]


@pytest.mark.parametrize("mode,fmt,m,n,red,us", SHORT_TIMES)
def test_short_reductions(plan, mode, fmt, m, n, red, us):
    _assert_no_slower_than_the_large_tile(plan, mode, fmt, m, n, red, 1, us)


E2M1_TIMES = [  # mode, rows, columns, reduction, groups
    (DENSE, 368, 16320, 6528, 1, (191.7, 205.4, 210.9, 221.7, 166.7)),
    (DENSE, 10832, 560, 6720, 1, (178.9, 193.7, 215.4, 224.5, 171.0)),
    (DENSE, 9296, 528, 1664, 1, (53.3, 60.0, 58.8, 57.8, 49.3)),
    (RAGGED_M, 10206, 384, 1536, 8, (45.4, 56.1, 52.4, 45.9, 35.3)),
    (RAGGED_M, 18958, 256, 1280, 32, (41.1, 49.2, 49.7, 52.5, 40.9)),
]


@pytest.mark.parametrize("mode,m,n,red,groups,us", E2M1_TIMES)
def test_e2m1_kernels(plan, mode, m, n, red, groups, us):
    """The E2M1 128 x 64 kernel runs two workgroups per CU, the uniform one three."""
    _assert_no_slower_than_the_large_tile(plan, mode, U.E2M1, m, n, red, groups, us)


@pytest.mark.parametrize("fmt,m,n,red,groups,us", RAGGED_M_TIMES)
def test_ragged_m_kernels(plan, fmt, m, n, red, groups, us):
    _assert_no_slower_than_the_large_tile(plan, RAGGED_M, fmt, m, n, red, groups, us)


@pytest.mark.parametrize("mode,m,n,red,groups", [
    (RAGGED_M, 1, 350080, 32, 1024),  # 1024 groups, one token: 3072 tile rows of 64, mostly of empty groups
    (RAGGED_M, 1000, 200064, 64, 2000),
    (DENSE, 1 << 20, 1 << 18, 32, 1),  # 2^24 tiles of 128 x 128, 2^26 of 64 x 64
    (RAGGED_K, 1 << 19, 1 << 17, 32, 2),
])
def test_mx_gemm_grids_stay_inside_a_launch(plan, mode, m, n, red, groups):
    tile, threads = mx_kernel(plan, mode, m, n, red, groups)
    assert threads < 1 << 32, tile


@pytest.mark.parametrize("n", [32, 64, 128])
@pytest.mark.parametrize("cols", [1, 1 << 29, (1 << 30) - 128, (1 << 31) - 1])
def test_wide_rht_quantizer_grids_stay_inside_a_launch(plan, n, cols):
    plan.ufp4_plan_cols_wide.restype = ctypes.c_int64
    assert 0 < plan.ufp4_plan_cols_wide(n, ctypes.c_int64(cols)) < 1 << 32


@pytest.mark.parametrize("mx,resident", [(0, 6), (1, 4)])
def test_grouped_quantizer_runs(plan, mx, resident):
    """Every tile in exactly one run, runs that differ by one tile at most, and no scan of the group offsets per tile or
    two once there is more than one round of workgroups (six or four to a CU)."""
    plan.ufp4_plan_grouped.restype = ctypes.c_int64
    longest = ctypes.c_int64()
    rnd = 256 * resident
    for tiles in (1, 2, 300, rnd - 1, rnd, rnd + 1, 6144, 8 * rnd, 8 * rnd + 1, 25000, 98305, (1 << 31) - 1):
        wg = plan.ufp4_plan_grouped(mx, ctypes.c_int64(tiles), ctypes.byref(longest))
        assert longest.value == -(-tiles // wg) and wg * 256 < 1 << 32
        assert wg == tiles if tiles <= rnd else wg % rnd == 0
        assert longest.value >= 4 or tiles < 4 * rnd  # 98304 tokens of 256 columns: 6144 tiles, four to a scan


# us on tiles and in the register kernel, each the mean of the same input again and of 1 GiB of inputs in turn; two operands
# of 80 to 100 Mi elements in a layer step of 160 tokens, a fifth of which they are
TILE_TIMES = [  # format, rounding, dual, rht, rows, cols, tile, register
    (U.UNIFORM, U.RTNE, 0, 1, 8192, 11008, 47.1, 48.3), (U.UNIFORM, U.RTNE, 0, 1, 24048, 4624, 63.8, 61.9),
    (U.UNIFORM, U.RTNE, 0, 1, 16384, 16384, 140.2, 135.7), (U.UNIFORM, U.RTNE, 0, 1, 32768, 16384, 280.4, 262.1),
    (U.UNIFORM, U.RTNE, 0, 0, 32768, 16384, 250.0, 261.1), (U.UNIFORM, U.SR, 0, 1, 4096, 8192, 26.0, 26.9),
    (U.UNIFORM, U.SR, 0, 1, 8192, 8192, 47.5, 45.9), (U.UNIFORM, U.SR, 0, 1, 8192, 11008, 62.9, 58.1),
    (U.UNIFORM, U.SR, 0, 0, 8192, 11008, 49.2, 49.7), (U.UNIFORM, U.SR, 0, 0, 16384, 16384, 148.0, 137.4),
    (U.E2M1, U.RTNE, 0, 1, 8192, 6144, 40.6, 42.3), (U.E2M1, U.RTNE, 0, 1, 8192, 11008, 70.2, 67.3),
    (U.E2M1, U.RTNE, 0, 0, 8192, 9216, 45.2, 47.3), (U.E2M1, U.RTNE, 0, 0, 16384, 16384, 153.6, 138.9),
    (U.E2M1, U.SR, 0, 1, 16384, 16384, 389.0, 397.8), (U.E2M1, U.SR, 0, 0, 24048, 4624, 146.9, 147.9),
    (U.E2M1, U.SR, 0, 0, 16384, 16384, 333.8, 321.1), (U.UNIFORM, U.RTNE, 1, 1, 8192, 9216, 62.3, 62.8),
    (U.UNIFORM, U.RTNE, 1, 1, 16224, 5520, 86.7, 93.3), (U.UNIFORM, U.RTNE, 1, 1, 8192, 11008, 88.4, 93.9),
    (U.UNIFORM, U.RTNE, 1, 1, 16384, 16384, 224.9, 203.4),
    (U.UNIFORM, U.RTNE, 1, 0, 16384, 12288, 140.8, 150.3), (U.UNIFORM, U.SR, 1, 1, 24048, 4624, 133.7, 141.0),
    (U.UNIFORM, U.SR, 1, 1, 16384, 16384, 306.5, 298.0), (U.E2M1, U.RTNE, 1, 1, 12288, 12288, 190.3, 193.3),
    (U.E2M1, U.RTNE, 1, 1, 32768, 16384, 667.2, 647.9), (U.E2M1, U.SR, 1, 1, 32768, 16384, 1422.6, 1533.0),
]


@pytest.mark.parametrize("fmt,rounding,dual,rht,rows,cols,tile,register", TILE_TIMES)
def test_quantizer_tiles_where_they_are_faster(plan, fmt, rounding, dual, rht, rows, cols, tile, register):
    plan.ufp4_plan_tile_most.restype = ctypes.c_int64
    tiles = rows * cols <= plan.ufp4_plan_tile_most(fmt, rounding, dual, rht)
    assert tiles == (tile < register)


@pytest.mark.parametrize("m,n,red,groups,a_rows,us", [  # us of the 256 x 256, 128 x 128 and 64 x 64 tiles
    (12759, 512, 2432, 64, 16384, (34.9, 33.7, 38.9)), (683, 512, 896, 64, 8320, (17.3, 12.2, 15.1)),
    (778, 2560, 896, 16, 2304, (18.5, 21.4, 19.6)), (3375, 2304, 512, 4, 3584, (15.4, 16.2, 16.2)),
    (9273, 1792, 256, 16, 10496, (25.2, 23.1, 26.5)), (48961, 384, 256, 4, 49152, (23.3, 18.7, 24.3)),
    (31445, 384, 1664, 8, 31872, (42.0, 29.6, 35.7)), (5267, 2688, 4096, 4, 5376, (86.0, 51.4, 83.2)),
    (17081, 1408, 2560, 32, 19200, (93.0, 74.7, 101.8)), (601, 256, 384, 128, 16384, (12.1, 8.9, 11.0)),
])
def test_mx_ragged_m_tiles(plan, m, n, red, groups, a_rows, us):
    tile, _ = mx_kernel(plan, RAGGED_M, m, n, red, groups, a_rows)
    assert us[(256, 128, 64).index(tile)] <= 1.04 * us[0], tile
