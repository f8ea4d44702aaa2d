"""Parity of the variants the planner picks by itself, on both sides of the
tile counts where its choice changes, against the FP64 oracle: rel-L2 <=
1e-6*log2(N) in complex64, 1e-3 (fp16) and 8e-3 (bf16) on the quantised input."""
import numpy as np
import pytest

import oracle
from paper_1707_07263_amd import capi, workloads
from gpu_helpers import from_gpu_16, quantised, rel_l2_rows, require_gpu, to_gpu_16, to_gpu_c64, tol_fp32

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

DTYPES = {"c64": capi.FFT_C64, "f16": capi.FFT_C16F, "bf16": capi.FFT_C16BF}


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def check(dev, shape, batch, dt, inverse, schedule=None):
    n = int(np.prod(shape))
    x = workloads.normal_batch(n, batch, seed=n % 1009 + batch).reshape([batch] + list(shape))
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16}.get(dt)
    xt = to_gpu_c64(x, dev) if dt == "c64" else to_gpu_16(x, dev, tdt)
    y = torch.empty_like(xt)
    h = capi.fft_plan_ex(list(shape), batch, len(shape), DTYPES[dt],
                         capi.FFT_INVERSE if inverse else capi.FFT_FORWARD, schedule)
    try:
        capi.fft_exec(h, xt.data_ptr(), y.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        capi.fft_destroy(h)
    xr = x.astype(np.complex64) if dt == "c64" else quantised(x, tdt)
    ref = (oracle.fft if len(shape) == 1 else oracle.fft2)(xr, inverse=inverse)
    got = y.cpu().numpy() if dt == "c64" else from_gpu_16(y)
    err = rel_l2_rows(got.reshape(batch, n), np.asarray(ref).reshape(batch, n), n).max()
    assert err <= {"c64": tol_fp32(n), "f16": 1e-3, "bf16": 8e-3}[dt], (shape, batch, dt, inverse, float(err))


# one line; a partial tile; for 1024 to 4096 points the last count below the
# persistent kernel (8 tiles for each of 256 CUs) and the first at it, plus a
# ragged tile; for the longest lines a persistent walk of more than one round
ROWS = [(n, b) for n in (2, 8, 16, 32, 64, 256, 512) for b in (1, 37)]
ROWS += [(4, 1000), (16, 1000), (32, 1001), (64, 4097)]  # short rows: whole tiles and a partial one
ROWS += [(1024, 1), (1024, 8188), (1024, 8189), (2048, 3), (2048, 4094), (2048, 4095), (4096, 1), (4096, 2047),
         (4096, 2048), (8192, 1), (8192, 259), (16384, 1), (16384, 259)]


@pytest.mark.parametrize("n,batch", ROWS)
@pytest.mark.parametrize("dt", sorted(DTYPES))
def test_rows(dev, n, batch, dt):
    for inverse in (False, True):
        check(dev, [n], batch, dt, inverse)


# batches around the tile counts where the passes' widths change: for a
# first or second pass of 1024 points 16 lines per tile need 256 tiles, for
# 256 points 32 lines 512; one transform runs the narrowest tiles
SPLITS = [(1 << 15, 1), (1 << 15, 33), (1 << 16, 1), (1 << 16, 31), (1 << 16, 65), (1 << 17, 1), (1 << 17, 9),
          (1 << 18, 1), (1 << 18, 3), (1 << 18, 17), (1 << 19, 1), (1 << 19, 5), (1 << 20, 1), (1 << 20, 3),
          (1 << 20, 5), (1 << 21, 1), (1 << 21, 5), (1 << 22, 1), (1 << 23, 1)]


@pytest.mark.parametrize("n,batch", SPLITS)
@pytest.mark.parametrize("dt", sorted(DTYPES))
def test_splits(dev, n, batch, dt):
    check(dev, [n], batch, dt, bool(batch & 2) or n == 1 << 22)


# every column length, few and many columns (fewer than the preferred tile is
# wide among them)
COLUMNS = [(1 << lg, c, b) for lg in range(1, 12) for c, b in ((4, 3), (64, 2))]
COLUMNS += [(512, 2048, 1), (1024, 1024, 3), (2048, 512, 3), (32, 4096, 5), (8192, 8, 1), (4096, 8, 2)]


@pytest.mark.parametrize("rows,cols,batch", COLUMNS)
@pytest.mark.parametrize("dt", sorted(DTYPES))
def test_columns(dev, rows, cols, batch, dt):
    for inverse in (False, True):
        check(dev, [rows, cols], batch, dt, inverse)


# lengths whose tiles are partly filled: fewer lines than a tile of 4096
# points holds, fewer columns than a strip is wide, second passes shorter and
# longer than the first, an item count on either side of the pairing by 16,
# every first-pass length down to 2 points
MANY = [[1], [2] * 5, [4096], [8192], [1 << 15], [1 << k for k in range(17)], [64] * 1025, [1 << 13] * 9,
        [1 << 16] * 3 + [8] * 7 + [1 << 12] * 2, [1 << 20, 1 << 14], [256, 1 << 17, 16]]


@pytest.mark.parametrize("sizes", MANY, ids=lambda s: f"{len(s)}x{max(s)}")
@pytest.mark.parametrize("schedule", [None, "flat=1;pass2=2", "flat=1;n1.13=1;n1.14=3;n1.16=12;n1.15=3"])
@pytest.mark.parametrize("dt", sorted(DTYPES))
def test_many_default_kernel(dev, sizes, schedule, dt):
    total = sum(sizes)
    x = workloads.normal_batch(total, 1, seed=total % 997)[0]
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16}.get(dt)
    xt = to_gpu_c64(x, dev) if dt == "c64" else to_gpu_16(x, dev, tdt)
    xr = x.astype(np.complex64) if dt == "c64" else quantised(x, tdt)
    for inverse in (False, True):
        h = capi.fft_plan_many_ex(sizes, DTYPES[dt], capi.FFT_INVERSE if inverse else capi.FFT_FORWARD, schedule)
        try:
            assert capi.fft_plan_info(h)["pass_variant"] == ["many_flat"]
            y = torch.empty_like(xt)
            capi.fft_exec(h, xt.data_ptr(), y.data_ptr(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
        finally:
            capi.fft_destroy(h)
        got = y.cpu().numpy() if dt == "c64" else from_gpu_16(y)
        ref = oracle.fft_many(xr, np.array(sizes), inverse=inverse)
        at = 0
        for n in sizes:
            err = rel_l2_rows(got[at:at + n], ref[at:at + n], n).max()
            assert err <= {"c64": tol_fp32(n), "f16": 1e-3, "bf16": 8e-3}[dt], (n, inverse, float(err))
            at += n


# images of 2048 rows and more through the Python layer: fused row passes of
# every row length, a batch of several images in one column launch, columns
# outside the rule, in place (by the plan's own exec too)
@pytest.mark.parametrize("rows,cols,batch", [(2048, 256, 3), (2048, 1024, 2), (2048, 2048, 1), (2048, 4096, 2),
                                             (4096, 512, 3), (4096, 2048, 1), (4096, 32, 3), (8192, 256, 2),
                                             (16384, 256, 1)])
@pytest.mark.parametrize("inverse", [False, True])
def test_images_by_rule(dev, rows, cols, batch, inverse):
    from paper_1707_07263_amd import api
    n = rows * cols
    x = workloads.normal_batch(n, batch, seed=rows + cols).reshape(batch, rows, cols)
    xt = to_gpu_c64(x, dev)
    ref = oracle.fft2(x.astype(np.complex64), inverse=inverse).reshape(batch, n)
    got = api.fft2(xt, inverse=inverse)
    assert rel_l2_rows(got.cpu().numpy().reshape(batch, n), ref, n).max() <= tol_fp32(n)
    y = xt.clone()
    api.fft2(y, inverse=inverse, out=y)
    assert torch.equal(y, got)
    api.clear_cache()
    plan = api.get_plan([rows, cols], batch, capi.FFT_C64, capi.FFT_INVERSE if inverse else capi.FFT_FORWARD)
    z = xt.clone()
    plan.exec(z, z)
    assert torch.equal(z, got)


# stage twiddles as products of two factors against the same butterflies with
# the stage table: a product is rounded once at its own size, like a table's
# entry, beside terms some 2^-3 of that, so the errors differ by about 1%
@pytest.mark.parametrize("shape,factors,table", [
    ([8192], "single=r8192p16w1q_c64", "single=r8192p16w1_c64"),
    ([64, 4096], "rowcol=4;row=f4096p16w4q_c64", "rowcol=4;row=f4096p16w4qx_c64"),
])
def test_factored_twiddles_are_as_good_as_tables(dev, shape, factors, table):
    n = int(np.prod(shape))
    batch = (1 << 20) // n
    x = workloads.normal_batch(n, batch, seed=5).reshape([batch] + shape).astype(np.complex64)
    xt = to_gpu_c64(x, dev)
    ref = (oracle.fft if len(shape) == 1 else oracle.fft2)(x)
    err = []
    for schedule in (factors, table):
        y = torch.empty_like(xt)
        h = capi.fft_plan_ex(shape, batch, len(shape), capi.FFT_C64, capi.FFT_FORWARD, schedule)
        try:
            capi.fft_exec(h, xt.data_ptr(), y.data_ptr(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
        finally:
            capi.fft_destroy(h)
        err.append(np.linalg.norm(y.cpu().numpy().ravel() - np.asarray(ref).ravel()))
    assert err[0] <= 1.01 * err[1], err
