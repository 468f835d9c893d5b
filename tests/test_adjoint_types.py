"""The adjoint kernels' reverse functions in both element types: on the host,
FP64 against the term-by-term form and FP32 against FP64; on the GPU the FP32
adjoint of a step against the FP64 one on the same data, through each kernel of
the y-pass."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_reverse_functions_in_both_types(tmp_path):
    hipcc = shutil.which('hipcc') or '/opt/rocm/bin/hipcc'
    if not os.path.exists(hipcc):
        pytest.skip('hipcc not available')
    exe = str(tmp_path / 'adjoint_types_check')
    subprocess.run([hipcc, '-O1', '-std=c++17', '--offload-arch=gfx950',
                    f'-I{os.path.join(ROOT, "paper_2411_11229_amd", "csrc")}',
                    os.path.join(ROOT, 'tests', 'cpu_math', 'adjoint_types_check.cpp'), '-o', exe],
                   check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    print(res.stdout)
    assert res.returncode == 0 and 'ALL OK' in res.stdout, res.stdout + res.stderr


@pytest.mark.gpu
@pytest.mark.parametrize('basis', ['cell', 'interface'])
@pytest.mark.parametrize('ends', [('periodic',) * 2, ('reflective', 'transmissive')], ids=lambda e: e[0][:5])
@pytest.mark.parametrize('system,nx,ny', [('euler', 200, 1), ('euler', 61, 40), ('euler', 128, 300),
                                          ('euler', 700, 800), ('burgers', 61, 40), ('burgers', 700, 800)])
def test_f32_adjoint_against_f64(system, nx, ny, ends, basis):
    """61x40 takes the y-pass with a wavefront per row in blocks of one row, 128x300
    in blocks of three and a remainder, 700x800 the marching one. Unrelated states from
    cell to cell, so that no differences cancel. The bound: each of about 64
    roundings between the inputs of a stage and its result acts like a change by
    2^-24 of the inputs (measured in FP64, over several such changes) or of the
    result; three stages, whose states are recomputed in FP32."""
    from paper_2411_11229_amd import hweno as H
    if system == 'burgers':
        if basis == 'interface':
            pytest.skip('scalar laws have one basis')
        ends = tuple('transmissive' if e == 'reflective' else e for e in ends)
    print(system, nx, ny, ends, basis, flush=True)
    dim = 1 if ny == 1 else 2
    rng = np.random.default_rng(nx + ny)
    shape = (ny, nx) if dim == 2 else (nx,)
    if system == 'burgers':
        U = rng.uniform(-1, 1, (1,) + shape)
    else:
        r, p = rng.uniform(1, 2, shape), rng.uniform(1, 2, shape)
        vel = [rng.uniform(-0.5, 0.5, shape) for _ in range(dim)]
        U = np.stack([r, *(r * v for v in vel), p / 0.4 + 0.5 * r * sum(v * v for v in vel)])
    nf = dim + 1
    X = [U] + [rng.uniform(-1, 1, U.shape) / 0.1 for _ in range(nf - 1)]
    lam = [rng.standard_normal(U.shape) for _ in range(nf)]
    single = lambda a: torch.tensor(a, dtype=torch.float32, device='cuda')
    X, lam = [single(a) for a in X], [single(a) for a in lam]
    dt = torch.full((1,), 1e-3, dtype=torch.float64, device='cuda')
    rec = torch.full((6,), 2.5, dtype=torch.float64, device='cuda')
    bc = (ends + ('periodic',) * 2) if dim == 1 else ends + ends
    kw = dict(dim=dim, nx=nx, ny=ny, dx=0.1, dy=0.12, system=system, bc=bc, basis=basis)

    def adjoint(precision, X, lam):
        s = H.Solver(H.Problem(precision=precision, **kw))
        cast = lambda a: a.to(s.prob.dtype).contiguous()
        out = [s.new_state() for _ in range(nf)]
        s.adjoint_step(*[cast(a) for a in X], *([None] * (3 - nf)), dt, rec, [cast(a) for a in lam], out)
        return [a.double() for a in out]

    unit = 2.0 ** -24
    gen = torch.Generator(device='cuda').manual_seed(5)
    change = lambda a: a.double() * (1 + unit * (2 * torch.rand(a.shape, generator=gen, dtype=torch.float64,
                                                               device='cuda') - 1))
    got, want = adjoint('f32', X, lam), adjoint('f64', X, lam)
    others = [adjoint('f64', [change(a) for a in X], [change(a) for a in lam]) for _ in range(8)]
    for f in range(nf):
        assert torch.isfinite(got[f]).all() and torch.isfinite(want[f]).all()
        moved = max(float((o[f] - want[f]).abs().max()) for o in others)
        err = float((got[f] - want[f]).abs().max())
        bound = 3 * 64 * (moved + unit * float(want[f].abs().max()))
        print(f'  field {f}: error {err:.2e}, bound {bound:.2e}, largest {float(want[f].abs().max()):.2e}')
        assert err <= bound
