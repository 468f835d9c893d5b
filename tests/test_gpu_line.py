"""1D steps: short lines run whole steps in one block, longer ones a launch per
stage, their maxima through one accumulator slot or, beyond 64 blocks, several.
A step whose stage states are asked for always takes a launch per stage: the two
routes agree bit for bit (the same arithmetic, so no tolerance), also around a
skipped step and a clipped one, and every recorded alpha is the maximum of the
spectral radius over the state it belongs to."""
import pytest
import torch

from paper_2411_11229_amd import hweno as H
from paper_2411_11229_amd import workloads as WL

pytestmark = pytest.mark.gpu

WALLS = ('reflective', 'transmissive', 'periodic', 'periodic')
KINDS = {
    'burgers': lambda n: (WL.random_smooth_1d(n, 'burgers', seed=51), {}),
    'euler': lambda n: (WL.euler1d_riemann_sine(n, seed=2009), {}),
    'walls': lambda n: (WL.with_bc(WL.random_smooth_1d(n, 'euler', seed=54), WALLS), {}),
    'interface': lambda n: (WL.random_smooth_1d(n, 'euler', seed=53), dict(basis='interface')),
}


@pytest.mark.parametrize('rule', ['production', 'fixed'])
@pytest.mark.parametrize('kind,n', [(k, n) for k in KINDS for n in (5, 60, 61, 480, 481, 960, 961)] +
                         [('euler', 3840), ('euler', 3841)])
def test_steps_match_stage_launches(kind, n, rule):
    print(kind, n, rule, flush=True)
    w, extra = KINDS[kind](n)
    s = H.Solver(H.Problem(**w.problem_kwargs(), **extra))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device='cuda')
    zeros = lambda *k: torch.zeros(*k, dtype=torch.float64, device='cuda')
    kw = dict(rule=rule, cfl=0.1, dt_fixed=0.01 * w.dx)
    steps = 67 if n <= 61 else 3       # more than one launch holds; else a few
    # the end time falls inside the last step but one: it is clipped, the last skipped
    U, V, t, dts = dev(w.U), dev(w.V), zeros(1), zeros(steps)
    s.steps(U, V, None, t, steps, dt_used=dts, **kw)
    t_end = float(dts[:steps - 2].sum() + 0.5 * dts[steps - 2])
    U, V, t, dts, rec = dev(w.U), dev(w.V), zeros(1), zeros(steps), zeros(steps, 6)
    s.steps(U, V, None, t, steps, t_end=t_end, dt_used=dts, alpha_rec=rec, **kw)
    Us, Vs, ts, dtss, recs = dev(w.U), dev(w.V), zeros(1), zeros(steps), zeros(steps, 6)
    nf = w.U.size
    stages = zeros(4 * nf)
    for k in range(steps):
        before = Us.clone()
        s.step(Us, Vs, None, ts, t_end, dt_used=dtss[k:k + 1], alpha_rec=recs[k], stages=stages, **kw)
        if k < steps - 1:
            for j, X in enumerate((before, stages[:nf].view_as(Us), stages[2 * nf:3 * nf].view_as(Us))):
                assert float(s.max_wavespeed(X)[0]) == float(recs[k, 2 * j]), (k, j)
    s.health()
    assert float(ts) == t_end and float(dtss[-1]) == 0.0
    for name, a, b in zip(('U', 'V', 't', 'dt', 'alphas'), (U, V, t, dts, rec), (Us, Vs, ts, dtss, recs)):
        assert torch.equal(a, b), name


def test_short_line_raises_the_health_flags():
    w, _ = KINDS['euler'](120)
    s = H.Solver(H.Problem(**w.problem_kwargs()))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device='cuda')
    U, V, t = dev(w.U), dev(w.V), torch.zeros(1, dtype=torch.float64, device='cuda')
    U[0, 37] = -1.0
    s.steps(U, V, None, t, 1, rule='fixed', dt_fixed=1e-6)
    with pytest.raises(H.HwenoError):
        s.health()
