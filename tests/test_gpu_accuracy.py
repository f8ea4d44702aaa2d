"""Error of the planner's own choices against 64 bits, complex64, normal data:
no more than one radix-16 sequence per length gives (16, 8 x 16, 16 x 16,
4 x 16 x 16 x 16; 4 x 16 x 16 and 8 x 16 x 16 in the two-pass and 2-D plans),
measured on 2^24 points as the bounds below.  Over the points of a test such an
error varies by less than 0.1 % with the data: 0.3 % is allowed."""
import pytest

from paper_1707_07263_amd import api

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_helpers import norms, require_gpu  # noqa: E402

SLACK = 1.003


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def rel(got, want):
    return (torch.linalg.vector_norm(norms((got - want).reshape(1, -1))) /
            torch.linalg.vector_norm(norms(want.reshape(1, -1)))).item()


def normal(shape, dev):
    g = torch.Generator(device=dev).manual_seed(17)
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=g, device=dev))


ROWS = [(16, 1 << 17, 6.1165e-8), (64, 1 << 15, 8.0233e-8), (128, 1 << 14, 8.7301e-8), (256, 1 << 13, 9.5086e-8),
        (1024, 2060, 1.0913e-7), (8192, 256, 1.2944e-7), (16384, 128, 1.3311e-7), (1 << 19, 8, 1.6788e-7),
        (1 << 20, 4, 1.7062e-7), (1 << 21, 2, 1.7463e-7), (1 << 21, 8, 1.7463e-7), (1 << 22, 4, 1.7877e-7),
        (1 << 23, 1, 1.8445e-7), (1 << 23, 2, 1.8443e-7), (1 << 24, 1, 1.8929e-7), (1 << 25, 1, 1.9648e-7)]


@pytest.mark.parametrize("n,batch,bound", ROWS)
def test_lines(dev, n, batch, bound):
    x = normal((batch, n), dev)
    assert rel(api.fft(x), torch.fft.fft(x.to(torch.complex128))) <= SLACK * bound


IMAGES = [(16, 16, 4096, None), (128, 128, 128, 1.2702e-7), (1024, 32, 64, 1.3648e-7), (1024, 1024, 16, 1.6088e-7),
          (2048, 128, 64, 1.4913e-7), (2048, 2048, 1, 1.6937e-7), (2048, 4096, 1, 1.7522e-7), (8192, 128, 4, 1.6233e-7)]


@pytest.mark.parametrize("rows,cols,batch,bound", IMAGES)
def test_images(dev, rows, cols, batch, bound):
    x = normal((batch, rows, cols), dev)
    want = torch.fft.fft2(x.to(torch.complex128))
    if bound is None:  # by the radix-16 variants themselves
        bound = rel(api.fft2(x, schedule="row=r16p16w256_c64;col=c16p16w16_c64"), want)
    assert rel(api.fft2(x), want) <= SLACK * bound


# the batched kernel: its own radices, the same bounds
@pytest.mark.parametrize("n,bound", [(16, 6.1165e-8), (128, 8.7301e-8), (256, 9.5086e-8), (1024, 1.0913e-7)])
def test_many(dev, n, bound):
    count = (1 << 20) // n
    x = normal((count, n), dev)
    got = api.fft_many(x.reshape(-1), [n] * count).reshape(count, n)
    assert rel(got, torch.fft.fft(x.to(torch.complex128))) <= SLACK * bound
