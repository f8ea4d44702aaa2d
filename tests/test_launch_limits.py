"""The largest transforms that fit the memory (288 GB) fit the launch limit of
2^32 - 1 lanes too, by the planner's own choices (host only)."""
import pytest

from paper_1707_07263_amd import capi

VARIANTS = {}


def variant(name):
    if not VARIANTS:
        for i in range(capi.fft_variant_count()):
            VARIANTS[capi.fft_variant_name(i)] = capi.fft_variant_describe(i)
    return VARIANTS[name]


def lanes(name, points):
    d = variant(name)
    if "q" in name.split("_")[0]:
        return 0  # persistent: a grid of resident workgroups
    return points // (d["L"] * d["W"]) * d["threads"]


@pytest.mark.parametrize("dtype", (capi.FFT_C64, capi.FFT_C16F, capi.FFT_C16BF))
@pytest.mark.parametrize("points", (1 << 34, 1 << 35))
def test_strided(dtype, points):
    for lg in range(5, 25):
        d = capi.fft_describe([1 << lg], points >> lg, 1, dtype)
        for name in d["names"]:
            assert lanes(name, points) < 1 << 32, (lg, name)
    for shape in ((16, 64), (32, 32), (64, 32), (16, 4096), (512, 512), (4096, 64)):
        d = capi.fft_describe(list(shape), points // (shape[0] * shape[1]), 2, dtype)
        for name in d["names"]:
            assert lanes(name, points) < 1 << 32, (shape, name)


def test_batched():
    # one launch of a workgroup per tile for 4096 x 4096 points, not for
    # 2^35 points in tiles of 4096
    for count, lanes_per_item in ((1 << 12, 512), (1 << 23, None)):
        q = capi.fft_describe_many_launches([4096] * count, capi.FFT_C16F)
        assert len(q) == 3 and q[2] == q[1]
        if lanes_per_item:
            assert q[1] == count
        else:
            assert q[1] == count // 2  # tiles of 8192 points, from the queue
    with pytest.raises(capi.FFTError):
        capi.fft_describe_many_launches([4096] * (1 << 23), capi.FFT_C16F, "flat=1")
