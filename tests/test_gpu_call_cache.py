"""Repeated calls through the Python layer find the plan of their own
signature: shape, storage type, direction, scale, schedule and lengths, also
after the tuner stored a schedule or the cache was cleared."""
import numpy as np
import pytest

import oracle
from paper_1707_07263_amd import api, autotune, workloads
from gpu_helpers import rel_l2_rows, require_gpu, to_gpu_c64, tol_fp32

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def test_signatures_do_not_mix(dev, tmp_path):
    n, b = 256, 6
    x = workloads.normal_batch(n, b, seed=5).astype(np.complex64)
    xt = to_gpu_c64(x, dev)
    fwd, inv = oracle.fft(x), oracle.fft(x, inverse=True)
    for _ in range(3):
        for kw, ref in (({}, fwd), ({"inverse": True}, inv), ({"inverse": 1, "scale": 1.0}, inv * n),
                        ({"scale": 2}, 2 * fwd), ({"schedule": "single=r256p16w16_c64"}, fwd),
                        ({"scale": np.float64(0.5)}, 0.5 * fwd)):
            got = api.fft(xt, **kw).cpu().numpy()
            assert rel_l2_rows(got, ref, n).max() <= tol_fp32(n), kw
        # the same points in another shape, and a strided view
        got = api.fft(xt.reshape(2 * b, n // 2)).cpu().numpy()
        assert rel_l2_rows(got, oracle.fft(x.reshape(2 * b, n // 2)), n // 2).max() <= tol_fp32(n)
        got = api.fft(xt[::2]).cpu().numpy()
        assert rel_l2_rows(got, fwd[::2], n).max() <= tol_fp32(n)
        got = api.fft2(xt.reshape(6, 16, 16)).cpu().numpy()
        assert rel_l2_rows(got.reshape(6, -1), oracle.fft2(x.reshape(6, 16, 16)).reshape(6, -1), n).max() <= tol_fp32(n)
        autotune.save({}, str(tmp_path / "tuned.json"))  # a new generation of schedules
        api.clear_cache()
    with pytest.raises(ValueError):
        api.fft(xt.cpu())
    with pytest.raises(ValueError):
        api.fft(xt, out=torch.empty(b, n + 1, dtype=xt.dtype, device=dev))


def test_many_lengths_by_value(dev):
    x = workloads.normal_batch(96, 1, seed=9).astype(np.complex64)[0]
    xt = to_gpu_c64(x, dev)
    sizes = [64, 32]
    for _ in range(2):
        for s in ([64, 32], [32, 64], (32, 32, 32), np.array([64, 32]), [64.0, 32.0]):
            got = api.fft_many(xt, s).cpu().numpy()
            at = 0
            for n in (int(v) for v in s):
                ref = oracle.fft(x[None, at:at + n])
                assert rel_l2_rows(got[None, at:at + n], ref, n).max() <= tol_fp32(n)
                at += n
    api.fft_many(xt, sizes)
    sizes[1] = 16  # the same list with other lengths: looked at again
    with pytest.raises(ValueError):
        api.fft_many(xt, sizes)
