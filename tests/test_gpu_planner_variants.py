"""Parity of every variant the planner picks by itself up to 2^24 points, at
the batches where its choice changes and the ones before them, against float64:
per transform rel-L2 <= 1e-6*log2(N) in complex64, 1e-3 (fp16) and 8e-3 (bf16)
on the stored input; the three-pass lengths in every storage type; and the
4096 x 4096 image in 16-bit storage by both of its plans."""
import math

import pytest

import planner_cases
from paper_1707_07263_amd import api
from gpu_helpers import norms, require_gpu, tol_fp32

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

STORAGE = {"c64": torch.complex64, "f16": torch.float16, "bf16": torch.bfloat16}


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def check(dev, shape, batch, dt, schedule=None):
    n = math.prod(shape)
    dims = (-2, -1) if len(shape) == 2 else (-1,)
    tol = {"c64": tol_fp32(n), "f16": 1e-3, "bf16": 8e-3}[dt]
    g = torch.Generator(device=dev).manual_seed(n % 1009 + batch)
    x = torch.randn((batch,) + tuple(shape) + (2,), generator=g, device=dev)
    x = torch.view_as_complex(x) if dt == "c64" else x.to(STORAGE[dt])

    def wide(t):
        return t.to(torch.complex128) if dt == "c64" else torch.view_as_complex(t.to(torch.float64))

    for inverse in (False, True):
        f = api.fft if len(shape) == 1 else api.fft2
        got = wide(f(x, inverse=inverse, schedule=schedule)).reshape(batch, n)
        name = "ifftn" if inverse else "fftn"
        ref = getattr(torch.fft, name)(wide(x), dim=dims).reshape(batch, n)
        err = (norms(got - ref) / norms(ref)).max().item()
        assert err <= tol, (shape, batch, dt, inverse, err)


CASES = [(dt, shape, batch) for dt, code in planner_cases.DTYPES.items()
         for shape, batch in planner_cases.lines(code) + planner_cases.images(code)]


def label(v):
    return "x".join(map(str, v)) if isinstance(v, tuple) else None


@pytest.mark.parametrize("dt,shape,batch", CASES, ids=label)
def test_choice(dev, dt, shape, batch):
    check(dev, shape, batch, dt)


@pytest.mark.parametrize("n", (1 << 25, 1 << 26))
@pytest.mark.parametrize("dt", sorted(STORAGE))
def test_three_passes(dev, n, dt):
    check(dev, (n,), 1, dt)


@pytest.mark.parametrize("schedule", ("col3=0", "col3=1"))
@pytest.mark.parametrize("dt", ("f16", "bf16"))
def test_16bit_4096x4096_image_by_both_plans(dev, dt, schedule):
    check(dev, (4096, 4096), 1, dt, schedule)
