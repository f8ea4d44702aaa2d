"""In-place 2-D transforms whose plan fuses the rows with a column step: the
results of the out-of-place call, to the bit, with no memory shared between
calls, streams or handles and none kept between calls."""
import numpy as np
import pytest

import oracle
from paper_1707_07263_amd import api, autotune, capi, workloads
from gpu_helpers import rel_l2_rows, require_gpu, to_gpu_c64, tol_fp32

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def image(rows, cols, batch, seed, dev):
    x = workloads.normal_batch(rows * cols, batch, seed=seed).reshape(batch, rows, cols)
    return to_gpu_c64(x, dev)


# by the rule (2048 rows and more) and by a tuned entry (4096 x 4096), with
# scratch from torch for each call and without
@pytest.mark.parametrize("scratch", [True, False])
@pytest.mark.parametrize("rows,cols,batch", [(2048, 256, 3), (2048, 2048, 5), (4096, 4096, 1)])
def test_two_streams(dev, rows, cols, batch, scratch, monkeypatch):
    if not scratch:
        monkeypatch.setattr(api, "_SCRATCH_MAX", 0)
    xs = [image(rows, cols, batch, seed, dev) for seed in (1, 2)]
    want = [api.fft2(x) for x in xs]
    streams = [torch.cuda.Stream(dev) for _ in xs]
    torch.cuda.synchronize()
    for _ in range(5):
        ys = [x.clone() for x in xs]
        torch.cuda.synchronize()
        for s, y in zip(streams, ys):
            with torch.cuda.stream(s):
                api.fft2(y, out=y)
        torch.cuda.synchronize()
        for y, w in zip(ys, want):
            assert torch.equal(y, w)


# cycles of the row shuffle: rotations of 11 to 14 bits by 1 and by 2, images
# down to the smallest (2 r rows) and more than one
@pytest.mark.parametrize("rows,cols,batch,schedule", [
    (2048, 2048, 2, None), (2048, 256, 1, None), (4096, 512, 1, None), (8192, 256, 3, None), (16384, 512, 1, None),
    (4096, 4096, 1, None), (4, 2048, 3, "rowcol=2"), (8, 256, 5, "rowcol=4"), (64, 512, 2, "rowcol=4"),
    (32, 4096, 2, "rowcol=2")])
@pytest.mark.parametrize("inverse", [False, True])
def test_without_scratch(dev, rows, cols, batch, schedule, inverse):
    n = rows * cols
    x = image(rows, cols, batch, rows + cols, dev)
    plan = api.get_plan([rows, cols], batch, capi.FFT_C64, capi.FFT_INVERSE if inverse else capi.FFT_FORWARD,
                        schedule=schedule)
    assert plan.info()["pass_variant"][0].startswith("f")
    want = torch.empty_like(x)
    stream = torch.cuda.current_stream().cuda_stream
    capi.fft_exec(plan.handle, x.data_ptr(), want.data_ptr(), stream)
    ref = oracle.fft2(x.cpu().numpy(), inverse=inverse).reshape(batch, n)
    assert rel_l2_rows(want.cpu().numpy().reshape(batch, n), ref, n).max() <= tol_fp32(n)
    # by the handle, by the allocation-free exec (above its limit for 1-D
    # plans, too), by the plan on a stream given by handle
    for run in (lambda y: capi.fft_exec(plan.handle, y.data_ptr(), y.data_ptr(), stream),
                lambda y: capi.fft_exec_static(plan.handle, y.data_ptr(), y.data_ptr(), stream),
                lambda y: plan.exec(y, y, stream=stream), lambda y: plan.exec(y, y)):
        y = x.clone()
        run(y)
        assert torch.equal(y, want)


def test_no_memory_is_kept(dev, monkeypatch):
    monkeypatch.setattr(api, "_SCRATCH_MAX", 64 << 20)
    for rows, cols, batch in ((2048, 1024, 1), (4096, 1024, 3)):
        y = image(rows, cols, batch, 3, dev)
        api.fft2(y, out=y)
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated(dev)
        torch.cuda.reset_peak_memory_stats(dev)
        api.fft2(y, inverse=True, out=y)
        torch.cuda.synchronize()
        assert torch.cuda.memory_allocated(dev) == before
        # a batch larger than the scratch allowed takes none at all
        extra = torch.cuda.max_memory_allocated(dev) - before
        assert extra <= (y.numel() * 8 if y.numel() * 8 <= api._SCRATCH_MAX else 0)


def test_under_capture(dev):
    x = image(2048, 512, 2, 4, dev)
    want = api.fft2(x)  # the plan exists; nothing has run in place yet
    y = x.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        api.fft2(y, out=y)
    for _ in range(4):
        y.copy_(x)
        junk = image(2048, 512, 2, 5, dev)
        api.fft2(junk, out=junk)  # eager work between the replays
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


def test_saved_fused_entry(dev, tmp_path, monkeypatch):
    monkeypatch.setattr(autotune, "_cache", dict(autotune._load_cache()))
    rows, cols = 2048, 1024
    schedule = "rowcol=4;xcd=10"
    autotune.save({autotune._key("plan", [rows, cols], 1, capi.FFT_C64): {"schedule": schedule}},
                  str(tmp_path / "tuned.json"))
    api.clear_cache()
    try:
        x = image(rows, cols, 1, 6, dev)
        want = api.fft2(x)
        plan = api.get_plan([rows, cols], 1, capi.FFT_C64, capi.FFT_FORWARD)
        y = x.clone()
        plan.exec(y, y)
        assert torch.equal(y, want)
    finally:
        api.clear_cache()
        autotune.generation += 1


def test_workspace_of_one_exec(dev):
    # 1-D, where the workspace is needed: this exec's own, and only if it is
    # large enough
    n, batch = 1 << 16, 3
    x = to_gpu_c64(workloads.normal_batch(n, batch, seed=8), dev)
    plan = api.get_plan([n], batch, capi.FFT_C64, capi.FFT_FORWARD)
    stream = torch.cuda.current_stream().cuda_stream
    want = torch.empty_like(x)
    capi.fft_exec(plan.handle, x.data_ptr(), want.data_ptr(), stream)
    need = capi.fft_workspace_size(plan.handle)
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    y = x.clone()
    for size in (0, need - 1):
        with pytest.raises(capi.FFTError):
            capi.fft_exec_ws(plan.handle, y.data_ptr(), y.data_ptr(), stream, ws.data_ptr(), size)
    with pytest.raises(capi.FFTError):
        capi.fft_exec_ws(plan.handle, y.data_ptr(), y.data_ptr(), stream, 0, need)
    assert torch.equal(y, x)
    capi.fft_exec_ws(plan.handle, y.data_ptr(), y.data_ptr(), stream, ws.data_ptr(), need)
    assert torch.equal(y, want)
