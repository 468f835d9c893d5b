"""A step call that returns an error between its launches leaves nothing behind
in the workspace: the next calls give what they give with a workspace of its
own, bit for bit. The error is a null event, which hipEventRecord refuses; the
state of the failed call has the larger wave speeds, so that a maximum left over
would be the next call's."""
import ctypes

import pytest
import torch

from paper_2411_11229_amd import hweno as H
from paper_2411_11229_amd import workloads as WL

pytestmark = pytest.mark.gpu


def _events(hip, bad):
    ev = (ctypes.c_void_p * 4)()
    for k in range(4):
        if k != bad:
            h = ctypes.c_void_p()
            assert hip.hipEventCreate(ctypes.byref(h)) == 0
            ev[k] = h
    return ev


@pytest.mark.parametrize('entry', ['step', 'steps'])
@pytest.mark.parametrize('bad', [0, 1, 2, 3])
@pytest.mark.parametrize('kind', ['1d', '1d_slots', 'tile', 'marcher'])
def test_nothing_is_left_by_a_failed_step(kind, bad, entry):
    print(kind, bad, entry, flush=True)
    # one accumulator slot, all slots, and the 2D kernels
    w = {'1d': lambda: WL.euler1d_riemann_sine(200, seed=2013),
         '1d_slots': lambda: WL.euler1d_riemann_sine(4000, seed=2013),
         'tile': lambda: WL.euler2d_smooth(64, seed=3400, ny=40, amp=0.02),
         'marcher': lambda: WL.euler2d_smooth(600, seed=3400, ny=500, amp=0.02)}[kind]()
    hip = ctypes.CDLL('libamdhip64.so')
    prob = H.Problem(**w.problem_kwargs())
    dev = lambda a: None if a is None else torch.tensor(a, dtype=torch.float64, device='cuda')
    state = lambda: [dev(w.U), dev(w.V), dev(w.W) if w.dim == 2 else None]
    zeros = lambda n: torch.zeros(n, dtype=torch.float64, device='cuda')

    def fail(s):
        X, ev = state(), _events(hip, bad)
        X[0][-1] *= 9.0                     # larger pressures
        t = zeros(1)
        with pytest.raises(H.HwenoError) as err:
            if entry == 'step':
                s.step(*X, t, events=ev)
            else:
                s.steps(*X, t, 1, events=ev)
        assert err.value.code == -3
        hip.hipGetLastError()
        torch.cuda.synchronize()
        for k in range(4):
            if ev[k]:
                hip.hipEventDestroy(ctypes.c_void_p(ev[k]))

    def two_steps(s):
        X, t, dts, rec = state(), zeros(1), zeros(2), zeros(12)
        s.steps(*X, t, 2, dt_used=dts, alpha_rec=rec, events=None)
        Y, t1, dt1, rec1 = state(), zeros(1), zeros(1), zeros(6)
        stages = torch.empty(2 * (w.dim + 1) * X[0].numel(), dtype=torch.float64, device='cuda')
        s.step(*Y, t1, dt_used=dt1, alpha_rec=rec1, stages=stages)   # (1D: a launch per stage)
        return [a for a in X + Y if a is not None] + [t, dts, rec, t1, dt1, rec1, stages]

    fresh, used = H.Solver(prob), H.Solver(prob)
    fail(used)
    assert used.max_wavespeed(dev(w.U)).tolist() == fresh.max_wavespeed(dev(w.U)).tolist()
    want = two_steps(H.Solver(prob))
    fail(used)
    # (a stage-wise step first: in 1D only those read the accumulators)
    Y, t1, rec1 = state(), zeros(1), zeros(6)
    stages = torch.empty(2 * (w.dim + 1) * Y[0].numel(), dtype=torch.float64, device='cuda')
    used.step(*Y, t1, alpha_rec=rec1, stages=stages)
    Z, t2, rec2 = state(), zeros(1), zeros(6)
    fresh.step(*Z, t2, alpha_rec=rec2, stages=torch.empty_like(stages))
    assert rec1.tolist() == rec2.tolist() and t1.tolist() == t2.tolist()
    fail(used)
    for a, b in zip(two_steps(used), want):
        assert torch.equal(a, b)
    used.health()
