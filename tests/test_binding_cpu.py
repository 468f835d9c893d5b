"""Python binding, no GPU: what it refuses before an address reaches the library."""
import pytest
import torch

from paper_2411_11229_amd import hweno as H


@pytest.mark.parametrize('device', ['cpu', 'meta'])
@pytest.mark.parametrize('dim', [1, 2])
def test_solver_refuses_devices_other_than_hip(device, dim):
    with pytest.raises(ValueError, match='HIP'):
        H.Solver(H.Problem(dim=dim, nx=32, ny=1 if dim == 1 else 16, dx=0.1, dy=0.1, system='euler'),
                 device=device)


class _HipTensor(torch.Tensor):
    """A host tensor that the argument checks take for a device one."""
    is_cuda = True
    device = property(lambda self: torch.device('cuda'))


class _Library:
    """Stands in for the library: every entry point succeeds without doing anything."""

    def __getattr__(self, name):
        return lambda *args: 0


CALLS = {
    'max_wavespeed': lambda s, X, sc: s.max_wavespeed(X[0], out=sc),
    'rhs': lambda s, X, sc: s.rhs(*X, alpha=sc),
    'step': lambda s, X, sc: s.step(*X, sc),
    'steps': lambda s, X, sc: s.steps(*X, sc, 2),
    'step_frozen': lambda s, X, sc: s.step_frozen(*X, sc, sc),
    'adjoint_step': lambda s, X, sc: s.adjoint_step(*X, sc, sc, X, X),
}


@pytest.mark.parametrize('change', [dict(precision='f32'), dict(nx=16), dict(ny=8), dict(system='burgers')],
                         ids=lambda c: next(iter(c)))
@pytest.mark.parametrize('call', CALLS)
def test_problem_changed_after_its_solver_was_made_is_refused(monkeypatch, call, change):
    """The library holds the problem as it was: outputs made for the changed one
    would be written out of range."""
    monkeypatch.setattr(H, 'load_library', lambda: _Library())
    monkeypatch.setattr(H, '_stream', lambda device: None)
    prob = H.Problem(dim=2, nx=32, ny=16, dx=0.1, dy=0.1, system='euler')
    s = H.Solver(prob, device='cpu')
    X = [torch.zeros(4, 16, 32, dtype=torch.float64).as_subclass(_HipTensor) for _ in range(3)]
    sc = torch.zeros(6, dtype=torch.float64).as_subclass(_HipTensor)
    CALLS[call](s, X, sc)
    for name, value in change.items():
        setattr(prob, name, value)
    with pytest.raises(ValueError):
        CALLS[call](s, X, sc)
