"""Calls that the Python layer refuses before any GPU work (no GPU needed)."""
import pytest

torch = pytest.importorskip("torch")

from paper_1707_07263_amd import api  # noqa: E402


def test_host_tensors_are_refused():
    x = torch.zeros(4, 16, dtype=torch.complex64)
    plan = object.__new__(api.Plan)  # no handle: nothing may be executed
    plan.handle, plan.workspace, plan.scratch = 0, None, 0
    for call in (lambda: api.fft(x), lambda: api.fft2(x, out=x), lambda: api.fft_many(x.reshape(-1), [32, 32]),
                 lambda: plan.exec(x, x), lambda: plan.exec(x, torch.empty_like(x))):
        with pytest.raises(ValueError):
            call()
