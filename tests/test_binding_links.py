"""Solver.update_links' checks of its arguments (no GPU: the library call and the
handle's counts are replaced)."""

import numpy as np
import pytest

L, D = 6, 2


@pytest.fixture
def solver(monkeypatch):
    from paper_1712_08288_amd import binding
    calls = []
    monkeypatch.setattr(binding, "_update_links", lambda h, q, u: calls.append((q, u)) or 0)
    monkeypatch.setattr(binding.Solver, "counts", lambda self: (40, L))
    sv = binding.Solver.__new__(binding.Solver)
    sv._h, sv.D = None, D
    sv.calls = calls
    return sv


def test_short_host_arrays_are_refused(solver):
    """The library reads L and L D values: no further than the array goes."""
    for kw in (dict(q=np.ones(L - 1)), dict(q=[]), dict(wall_u=np.zeros((L - 1, D))),
               dict(q=np.ones(L), wall_u=np.zeros(L))):
        with pytest.raises(ValueError):
            solver.update_links(**kw)
    assert not solver.calls
    solver.update_links(np.ones(L), np.zeros((L, D)))
    solver.update_links([0.5] * L)
    solver.update_links(np.ones(L + 3))      # what lies behind is not read
    solver.update_links()
    assert len(solver.calls) == 4 and solver.calls[3] == (None, None)


class DeviceTensor:
    """What update_links asks of a device tensor."""
    is_cuda, dtype = True, "torch.float64"

    def __init__(self, n, contiguous=True):
        self.n, self.contiguous = n, contiguous

    def numel(self):
        return self.n

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return 4096


def test_device_tensors_longer_than_the_links_are_taken(solver):
    """As host arrays are, and as they were when the autograd function brought
    device tensors to the host."""
    solver.update_links(DeviceTensor(L + 2), DeviceTensor(L * D + 1))
    assert [p.value for p in solver.calls[0]] == [4096, 4096]
    for t in (DeviceTensor(L - 1), DeviceTensor(L, contiguous=False)):
        with pytest.raises(ValueError):
            solver.update_links(t)
    assert len(solver.calls) == 1
