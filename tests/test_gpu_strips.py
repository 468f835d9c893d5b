"""The 2D forward stage kernels choose how many rows a block takes, and in
FP64 whether its rows go through one wavefront or one each; no choice may
change a result. Small grids (last strips of one row, of fewer rows than the
others, one strip for everything; the last column block ragged, or full; the
most rows that a block takes at once, and the first grid beyond) with every
kind of boundary, the source, both bases and a scalar law: the
operator and one step, the kernels' own choice against forced strip heights,
bit for bit (the rows' arithmetic is the same, so no tolerance)."""
import pytest
import torch

from paper_2411_11229_amd import hweno as H
from paper_2411_11229_amd import workloads as WL

pytestmark = pytest.mark.gpu


def _workload(kind, nx, ny):
    if kind == 'rayleigh-taylor':                 # walls, fixed states, source
        return WL.rayleigh_taylor(nx), {}
    if kind == 'double-mach':                     # fixed, transmissive and split sides
        return WL.double_mach(4 * nx), {}
    if kind == 'burgers':
        w = WL.paper_burgers2d(nx)
        return w, {}
    if kind == 'interface':
        return WL.euler2d_smooth(nx, seed=3100, ny=ny), dict(basis='interface')
    if kind == 'walls':
        w = WL.euler2d_smooth(nx, seed=3101, ny=ny)
        return WL.with_bc(w, ('reflective', 'transmissive', 'reflective', 'reflective')), {}
    return WL.euler2d_quadrants(nx, seed=4001, ny=ny), {}


CASES = [('quadrants', 61, 37), ('quadrants', 121, 250), ('quadrants', 6, 5),
         ('quadrants', 300, 301), ('quadrants', 300, 307), ('interface', 384, 251), ('walls', 384, 257),
         ('quadrants', 300, 408), ('quadrants', 300, 409), ('interface', 60, 41), ('walls', 59, 23), ('rayleigh-taylor', 40, None), ('double-mach', 34, None),
         ('burgers', 70, None)]


@pytest.mark.parametrize('precision', ['f64', 'f32'])
@pytest.mark.parametrize('kind,nx,ny', CASES, ids=[f'{c[0]}-{c[1]}x{c[2]}' for c in CASES])
def test_rows_per_block_leave_results_bit_identical(kind, nx, ny, precision):
    w, extra = _workload(kind, nx, ny)
    dtype = torch.float64 if precision == 'f64' else torch.float32
    s = H.Solver(H.Problem(**w.problem_kwargs(), precision=precision, **extra))
    dev = lambda a: torch.tensor(a, dtype=dtype, device='cuda')
    U0, V0, W0 = dev(w.U), dev(w.V), dev(w.W)
    alpha = s.max_wavespeed(U0)
    results = {}
    try:
        for rows in (0, 1, 2, 5, 7, w.ny):
            print(f'{w.name} {w.nx}x{w.ny} {precision} rows {rows or "auto"}', flush=True)
            H.set_strip_rows(rows)
            out = list(s.rhs(U0, V0, W0, alpha))
            U, V, W = U0.clone(), V0.clone(), W0.clone()
            t = torch.zeros(1, dtype=torch.float64, device='cuda')
            rec = torch.zeros(2, 6, dtype=torch.float64, device='cuda')
            s.steps(U, V, W, t, 2, cfl=0.1, alpha_rec=rec)
            torch.cuda.synchronize()
            results[rows] = out + [U, V, W, t, rec]
    finally:
        H.set_strip_rows(0)
    assert all(torch.isfinite(x).all() for x in results[0])
    for rows, got in results.items():
        for name, a, b in zip(('L1', 'L2', 'L3', 'vtilde', 'wtilde', 'U', 'V', 'W', 't', 'alphas'),
                              results[0], got):
            assert torch.equal(a, b), f'{name} differs between auto and {rows} rows'
