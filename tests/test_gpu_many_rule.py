"""Batches of long lengths, which take the queue kernel by rule: its queue
state is each call's own."""
import numpy as np
import pytest

import oracle
from paper_1707_07263_amd import api, capi, workloads
from gpu_helpers import rel_l2_rows, require_gpu, to_gpu_c64, tol_fp32

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [1 << 20, 1, 1 << 19, 8, 1 << 20, 64, 1 << 18, 1 << 20, 2]


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def packed(seed, dev):
    return to_gpu_c64(workloads.normal_batch(sum(SIZES), 1, seed=seed)[0], dev)


def test_two_streams(dev):
    plan = api.get_many_plan(SIZES, capi.FFT_C64, capi.FFT_FORWARD)
    assert plan.info()["pass_variant"] == ["many_2launch"]
    xs = [packed(seed, dev) for seed in (1, 2)]
    want = [api.fft_many(x, SIZES) for x in xs]
    for x, w in zip(xs, want):
        ref = oracle.fft_many(x.cpu().numpy(), np.array(SIZES))
        at, got = 0, w.cpu().numpy()
        for n in SIZES:
            assert rel_l2_rows(got[at:at + n], ref[at:at + n], n).max() <= tol_fp32(n), n
            at += n
    streams = [torch.cuda.Stream(dev) for _ in xs]
    outs = [torch.empty_like(x) for x in xs]
    torch.cuda.synchronize()
    for _ in range(8):
        for s, x, o in zip(streams, xs, outs):
            with torch.cuda.stream(s):
                o.zero_()
                api.fft_many(x, SIZES, out=o)
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert torch.equal(o, w)


def test_under_capture(dev):
    x = packed(3, dev)
    want = api.fft_many(x, SIZES)
    out = torch.empty_like(x)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        api.fft_many(x, SIZES, out=out)
    for _ in range(4):
        out.zero_()
        api.fft_many(x, SIZES)  # eager work between the replays
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
