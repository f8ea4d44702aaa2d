"""Which kernel a batched plan takes by itself (host only): the plain grid's
tiles hold 4096 points (512 lanes by 8), the persistent queue kernel's 8192."""
import random

import pytest

from paper_1707_07263_amd import capi

DTYPES = (capi.FFT_C64, capi.FFT_C16F, capi.FFT_C16BF)


def plain(sizes, dtype):
    """Whether the plan splits the batch as the plain grid does."""
    auto = [capi.fft_describe_many_launches(sizes, dtype, s).tolist() for s in (None, "flat=1", "pipe=2")]
    assert auto[1] != auto[2] and auto[0] in auto[1:]
    return auto[0] == auto[1]


def mixed(lo, hi, count):
    r = random.Random(lo * 100 + hi)
    return [1 << r.randint(lo, hi) for _ in range(count)]


@pytest.mark.parametrize("dtype", DTYPES)
def test_short_lengths_take_the_plain_grid(dtype):
    for sizes in ([64] * 3000, [1 << 13] * 64, [1 << 16] * 256, mixed(8, 16, 512), mixed(4, 16, 2000),
                  mixed(10, 18, 100), mixed(14, 18, 60), [1 << 20], [1 << 18] * 4, [1 << 20, 1 << 14]):
        assert plain(sizes, dtype), (len(sizes), max(sizes))


def test_long_lengths_take_the_queue():
    for sizes in ([1 << 18] * 64, [1 << 19] * 16, [1 << 20] * 4, [1 << 21], [1 << 22], mixed(0, 20, 160),
                  mixed(6, 20, 160), mixed(0, 16, 2000)):
        assert not plain(sizes, capi.FFT_C64), (len(sizes), max(sizes))
    for dtype in DTYPES[1:]:  # 16-bit passes gain less from wide strips
        for sizes in ([1 << 20] * 16, [1 << 22] * 4, mixed(0, 20, 160)):
            assert not plain(sizes, dtype), (len(sizes), max(sizes))
        for sizes in ([1 << 18] * 64, [1 << 20] * 4, mixed(6, 20, 160), mixed(0, 16, 2000)):
            assert plain(sizes, dtype), (len(sizes), max(sizes))
    # a kernel asked for by name is that kernel
    assert plain([64] * 3000, capi.FFT_C64)
    auto, flat = (capi.fft_describe_many_launches([1 << 20] * 4, capi.FFT_C64, s).tolist() for s in (None, "flat=1"))
    assert auto != flat
