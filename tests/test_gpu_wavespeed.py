"""max_wavespeed: one launch whose last block collects the maxima. One block,
two, as many as a launch has, and more cells than those take at once; larger
values first, so that a maximum left over from an earlier call would show; and
the first step's seed, which shares the accumulators, in between."""
import numpy as np
import pytest
import torch

from paper_2411_11229_amd import hweno as H
from paper_2411_11229_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('nx,ny', [(5, 5), (16, 16), (257, 1), (1024, 256), (700, 500)])
def test_max_wavespeed_of_successive_states(nx, ny):
    print(nx, ny, flush=True)
    if ny == 1:
        w = WL.euler1d_riemann_sine(nx, seed=2011)
    else:
        w = WL.euler2d_smooth(nx, seed=3300, ny=ny, amp=0.02)
    s = H.Solver(H.Problem(**w.problem_kwargs()))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device='cuda')
    g = 1.4
    for scale in (3.0, 1.0, 2.0):      # the energy times scale: other pressures
        U = w.U.copy()
        U[-1] *= scale
        vel = [U[1 + k] / U[0] for k in range(w.dim)]
        p = (g - 1.0) * (U[-1] - 0.5 * U[0] * sum(v * v for v in vel))
        c = np.sqrt(g * p / U[0])
        want = [float((np.abs(v) + c).max()) for v in vel] + [0.0] * (2 - w.dim)
        X = [dev(U), dev(w.V)] + ([dev(w.W)] if w.dim == 2 else [None])
        for _ in range(2):
            got = s.max_wavespeed(X[0]).cpu().numpy()
            # reciprocal and inverse root within two units, a few roundings
            assert np.abs(got - want).max() <= 1e-14 * max(want)
        t, rec = dev(np.zeros(1)), dev(np.zeros(6))
        s.step(*X, t, rule='fixed', dt_fixed=1e-6, alpha_rec=rec)
        assert rec.cpu().numpy()[:w.dim].tolist() == got[:w.dim].tolist()
