"""Python binding, no GPU: a workspace on a device without HIP streams is refused
before its address reaches the library."""
import pytest

from paper_2411_11229_amd import hweno as H


@pytest.mark.parametrize('device', ['cpu', 'meta'])
@pytest.mark.parametrize('dim', [1, 2])
def test_solver_refuses_devices_other_than_hip(device, dim):
    with pytest.raises(ValueError, match='HIP'):
        H.Solver(H.Problem(dim=dim, nx=32, ny=1 if dim == 1 else 16, dx=0.1, dy=0.1, system='euler'),
                 device=device)
