"""Host-side checks of the planner's own choices (no GPU): whatever the shape,
batch and storage type, the passes it picks cover the transform, their tiles
are no wider than their lines, and what could be planned before still can."""
import re

import pytest

from paper_1707_07263_amd import capi

DTYPES = (capi.FFT_C64, capi.FFT_C16F, capi.FFT_C16BF)
NAME = re.compile(r"([ractf])(\d+)p(\d+)w(\d+)")
BATCHES = (1, 2, 3, 5, 31, 64, 255, 256, 4099, 1 << 16)


def parse(name):
    m = NAME.match(name)
    return m.group(1), int(m.group(2)), int(m.group(4))


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lg", range(1, 25))
def test_1d(dtype, lg):
    n = 1 << lg
    for batch in BATCHES:
        d = capi.fft_describe([n], batch, 1, dtype)
        p = [parse(x) for x in d["names"]]
        if lg <= 14:
            assert len(p) == 1 and p[0][:2] == ("r", n)
            continue
        (ra, la, wa), (rb, lb, wb) = p
        assert (ra, rb) == ("a", "c") and la * lb == n and d["split"] == [la, lb]
        assert wa <= lb and wb <= la
        # a schedule that names the pass order explicitly plans the same way
        assert capi.fft_describe([n], batch, 1, dtype, f"split={la}")["names"] == d["names"]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lg_r", range(0, 15))
def test_2d(dtype, lg_r):
    for lg_c in range(0, 15):
        r, c = 1 << lg_r, 1 << lg_c
        for batch in (1, 3, 64):
            names = capi.fft_describe([r, c], batch, 2, dtype)["names"]
            p = [parse(x) for x in names if x != "copy_scale"]
            rows = [x for x in p if x[0] == "r"]
            cols = [x for x in p if x[0] in "ct"]
            assert [x[1] for x in rows] == ([c] if c > 1 else [])
            length = 1
            for x in cols:
                length *= x[1]
            assert length == r or (not cols and r == 1)
            # a column tile is wider than the columns only where no variant
            # is narrower
            for role, L, w in cols:
                if w > c:
                    widths = [capi.fft_variant_describe(i)["W"] for i in range(capi.fft_variant_count())
                              if capi.fft_variant_describe(i)["role"] == 2
                              and capi.fft_variant_describe(i)["L"] == L
                              and capi.fft_variant_describe(i)["dtype"] == dtype]
                    assert min(widths) > c, (r, c, names)


@pytest.mark.parametrize("dtype", DTYPES)
def test_2d_rule_plans_wherever_it_applies(dtype):
    from paper_1707_07263_amd import autotune
    ruled = 0
    for lg_r in range(0, 15):
        for lg_c in range(0, 15):
            r, c = 1 << lg_r, 1 << lg_c
            s = autotune.rule_for([r, c], dtype)
            if s is None:
                continue
            ruled += 1
            for batch in (1, 3, 1000):
                d = capi.fft_describe([r, c], batch, 2, dtype, s)
                p = [parse(x) for x in d["names"]]
                assert d["passes"] == 2 and p[0][1] == c
                assert p[0][0] == ("f" if "rowcol" in s else "r")
                # what the fused row pass leaves of the columns
                assert p[1][0] == "c" and p[1][1] * (p[0][2] if p[0][0] == "f" else 1) == r
    assert ruled > 0
