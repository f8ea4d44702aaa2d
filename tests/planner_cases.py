"""Shapes on both sides of every change of the planner's own choice (not
collected by pytest)."""
from paper_1707_07263_amd import autotune, capi

MAX_POINTS = 1 << 24
DTYPES = {"c64": capi.FFT_C64, "f16": capi.FFT_C16F, "bf16": capi.FFT_C16BF}


def plan_names(shape, batch, dtype):
    """Variants of the plan the Python layer asks for, without tuned entries."""
    schedule = autotune.rule_for(shape, dtype, batch) if len(shape) == 2 else None
    return tuple(capi.fft_describe(list(shape), batch, len(shape), dtype, schedule)["names"])


def steps(shape, dtype):
    """(batch, names) for the first batch of each choice and the last one
    before it, over batches up to MAX_POINTS points."""
    points = 1
    for n in shape:
        points *= n
    last = max(1, MAX_POINTS // points)
    grid = sorted({b for k in range(25) for b in ((1 << k) - 1, 1 << k, 3 << k) if 1 <= b <= last} | {last})
    out = {}
    names = {b: plan_names(shape, b, dtype) for b in grid}
    for lo, hi in zip(grid, grid[1:]):
        if names[lo] == names[hi]:
            continue
        a, c = lo, hi
        while c - a > 1:
            mid = (a + c) // 2
            if plan_names(shape, mid, dtype) == names[lo]:
                a = mid
            else:
                c = mid
        out[a], out[c] = names[lo], plan_names(shape, c, dtype)
    if not out:
        out[last] = names[last]
    return sorted(out.items())


def lines(dtype):
    """1-D cases: every step of every length up to 2^24."""
    return [((1 << lg,), b) for lg in range(1, 25) for b, _ in steps((1 << lg,), dtype)]


def images(dtype):
    """2-D cases: of the steps of all shapes, those with a choice (role and
    variant) that neither the lines nor an earlier image had."""
    seen = {n for shape, b in lines(dtype) for n in plan_names(shape, b, dtype)}
    out = []
    for lg_r in range(1, 14):
        for lg_c in range(1, 14):
            shape = (1 << lg_r, 1 << lg_c)
            for b, names in steps(shape, dtype):
                if b << (lg_r + lg_c) <= MAX_POINTS and not seen.issuperset(names):
                    seen.update(names)
                    out.append((shape, b))
    return out
