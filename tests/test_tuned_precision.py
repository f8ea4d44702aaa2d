"""16-bit batches: a length that fits a tile (up to 2^12 points) is transformed
in one pass, with nothing stored in between, by every stored schedule and by
everything the tuner may choose (host only)."""
import pytest

from paper_1707_07263_amd import autotune, capi, workloads

SIZES = [1 << lg for lg in range(1, 17)]


def two_pass_lengths(sizes, dtype, schedule):
    _, first_len, _ = capi.fft_describe_many(sizes, dtype, schedule)
    return {n for n, n1 in zip(sizes, first_len) if n1}


@pytest.mark.parametrize("dtype", (capi.FFT_C16F, capi.FFT_C16BF))
def test_one_pass_where_it_fits(dtype):
    long = {n for n in SIZES if n > 4096}
    stored = autotune.many_schedule_for([int(n) for n in workloads.uneven_sizes(512, 8, 16, seed=3)], dtype)
    assert stored is not None
    planned = 0
    for schedule in [None, stored] + autotune._many_grid(dtype):
        try:
            split = two_pass_lengths(SIZES, dtype, schedule)
        except capi.FFTError:  # a kernel that this storage type does not have
            assert schedule not in (None, stored)
            continue
        planned += 1
        assert split == long, schedule
    assert planned > 3
    for lg in range(1, 17):
        for key, value in autotune._length_options(lg, 13, 12, dtype):
            schedule = f"flat=1;pass2=13;{key}.{lg}={value}"
            assert two_pass_lengths(SIZES, dtype, schedule) == long, schedule


def test_complex64_may_split_any_length():
    assert ("pass", 2) in autotune._length_options(10, 13, 12, capi.FFT_C64)
    assert any("pass2=9" in s for s in autotune._many_grid(capi.FFT_C64))
