"""The cases of test_gpu_planner_variants reach every variant that the planner
picks by itself (host only)."""
import pytest

import planner_cases
from paper_1707_07263_amd import capi


@pytest.mark.parametrize("dt", sorted(planner_cases.DTYPES))
def test_every_default_variant_has_a_case(dt):
    dtype = planner_cases.DTYPES[dt]
    cases = planner_cases.lines(dtype) + planner_cases.images(dtype)
    tested = {n for shape, batch in cases for n in planner_cases.plan_names(shape, batch, dtype)}
    for lg in range(1, 25):
        last = planner_cases.MAX_POINTS >> lg
        for batch in {*range(1, min(last, 130) + 1), *(last * k // 97 for k in range(1, 98))} - {0}:
            names = planner_cases.plan_names((1 << lg,), batch, dtype)
            assert tested.issuperset(names), (lg, batch, names)
    for lg_r in range(1, 14):
        for lg_c in range(1, 14):
            last = max(1, planner_cases.MAX_POINTS >> (lg_r + lg_c))
            for batch in {1, 2, 3, 5, 17, 100, last // 3, last // 2, last} & set(range(1, last + 1)):
                if batch << (lg_r + lg_c) <= planner_cases.MAX_POINTS:
                    names = planner_cases.plan_names((1 << lg_r, 1 << lg_c), batch, dtype)
                    assert tested.issuperset(names), (lg_r, lg_c, batch, names)


def test_the_cases_are_the_steps():
    # 1024-point rows in complex64 turn persistent at 2048 tiles of 4 rows
    assert ((1024,), 8188) in planner_cases.lines(capi.FFT_C64)
    assert ((1024,), 8189) in planner_cases.lines(capi.FFT_C64)


def test_4096_rows_few_columns_keep_the_three_passes():
    # from one strip of columns per other CU on: rows, then whole columns
    for dt, most in (("c64", 128), ("f16", 256), ("bf16", 256)):
        dtype = planner_cases.DTYPES[dt]
        for cols in (16, 32, 64, 128):
            few, many = most // cols, most // cols + 1
            assert len(planner_cases.plan_names((4096, cols), few, dtype)) == 3
            assert len(planner_cases.plan_names((4096, cols), many, dtype)) == 2


def test_16384_point_rows_by_lines_per_cu():
    # one line per CU and more: fp16 changes its lanes, bf16 does not
    for dt, few in (("f16", "r16384p16w1_f16"), ("bf16", "r16384p32w1x_bf16")):
        names = [planner_cases.plan_names((16384,), b, planner_cases.DTYPES[dt]) for b in (1, 256, 257, 1024)]
        assert names == [(few,), (few,), (f"r16384p32w1x_{dt}",), (f"r16384p32w1x_{dt}",)]


def test_fewer_columns_than_any_tile_take_the_narrowest():
    # 16-bit columns have no tiles of 2 or 4: no more than half a tile idle
    # where a narrower one exists
    for dt in ("f16", "bf16"):
        dtype = planner_cases.DTYPES[dt]
        for rows, width in ((256, 8), (512, 8), (1024, 8), (2048, 4), (4096, 4)):
            for cols in (2, 4):
                for batch in (1, 64, 1024):
                    names = planner_cases.plan_names((rows, cols), batch, dtype)
                    d = {capi.fft_variant_name(i): i for i in range(capi.fft_variant_count())}
                    assert capi.fft_variant_describe(d[names[-1]])["W"] == width, names
