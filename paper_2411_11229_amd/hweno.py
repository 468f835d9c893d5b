"""Python binding of ``libhweno.so`` (the HWENO-I C ABI, include/hweno.h).

Argument marshalling only: every step of the scheme runs in the HIP kernels.
Tensors are torch tensors on the HIP device, contiguous, float64 or float32
(matching ``Problem.precision``), shaped ``[ncomp, nx]`` in 1D and
``[ncomp, ny, nx]`` in 2D. Work is enqueued on torch's current stream.

The library is loaded on first use; a missing library raises RuntimeError
(there is no CPU fallback).
"""
import ctypes
import os
from dataclasses import dataclass

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, 'libhweno.so')

SYSTEMS = {'advection': 0, 'burgers': 1, 'euler': 2}
BCS = {'periodic': 0, 'transmissive': 1, 'reflective': 2, 'dirichlet': 3, 'split': 4}
PRECISIONS = {'f64': 0, 'f32': 1}
BASES = {'cell': 0, 'interface': 1}
DT_RULES = {'production': 0, 'accuracy': 1, 'fixed': 2}
STATUS = {0: 'ok', -1: 'invalid argument', -2: 'unsupported', -3: 'HIP runtime error',
          -4: 'non-finite state', -5: 'non-physical state',
          -6: 'problem exceeds the static scratch'}


class HwenoError(RuntimeError):
    def __init__(self, code, what):
        super().__init__(f'{what}: {STATUS.get(code, code)} (status {code})')
        self.code = code


class _CSplit(ctypes.Structure):
    _fields_ = [('x0', ctypes.c_double), ('slope', ctypes.c_double), ('speed', ctypes.c_double),
                ('kind', ctypes.c_int32 * 2), ('state', (ctypes.c_double * 4) * 2)]


class _CProblem(ctypes.Structure):
    _fields_ = [('dim', ctypes.c_int32), ('nx', ctypes.c_int32), ('ny', ctypes.c_int32),
                ('dx', ctypes.c_double), ('dy', ctypes.c_double), ('system', ctypes.c_int32),
                ('adv_a', ctypes.c_double), ('adv_b', ctypes.c_double),
                ('gas_gamma', ctypes.c_double), ('gamma0', ctypes.c_double),
                ('d0', ctypes.c_double), ('eps', ctypes.c_double),
                ('bc', ctypes.c_int32 * 4), ('precision', ctypes.c_int32),
                ('char_basis', ctypes.c_int32), ('bc_state', (ctypes.c_double * 4) * 4),
                ('gravity', ctypes.c_double), ('split', _CSplit * 2)]


_P = ctypes.c_void_p
_SIGS = {
    'hweno_status_string': ([ctypes.c_int], ctypes.c_char_p),
    'hweno_workspace_bytes': ([ctypes.POINTER(_CProblem), ctypes.POINTER(ctypes.c_size_t)], ctypes.c_int),
    'hweno_workspace_init': ([ctypes.POINTER(_CProblem), _P, _P], ctypes.c_int),
    'hweno_max_wavespeed': ([ctypes.POINTER(_CProblem), _P, _P, _P, _P], ctypes.c_int),
    'hweno_rhs': ([ctypes.POINTER(_CProblem)] + [_P] * 11, ctypes.c_int),
    'hweno_step': ([ctypes.POINTER(_CProblem), _P, _P, _P, ctypes.c_int32, ctypes.c_double,
                    ctypes.c_double, ctypes.c_double, _P, _P, _P, _P, _P, _P], ctypes.c_int),
    'hweno_step_profiled': ([ctypes.POINTER(_CProblem), _P, _P, _P, ctypes.c_int32, ctypes.c_double,
                             ctypes.c_double, ctypes.c_double, _P, _P, _P, _P, _P, _P, _P],
                            ctypes.c_int),
    'hweno_steps': ([ctypes.POINTER(_CProblem), _P, _P, _P, ctypes.c_int32, ctypes.c_int32,
                     ctypes.c_double, ctypes.c_double, ctypes.c_double, _P, _P, _P, _P, _P, _P],
                    ctypes.c_int),
    'hweno_set_strip_rows': ([ctypes.c_int32], ctypes.c_int),
    'hweno_step_noalloc': ([ctypes.POINTER(_CProblem), _P, _P, _P, ctypes.c_int32, ctypes.c_double,
                            ctypes.c_double, ctypes.c_double, _P, _P, _P, _P], ctypes.c_int),
    'hweno_step_frozen': ([ctypes.POINTER(_CProblem)] + [_P] * 11, ctypes.c_int),
    'hweno_adjoint_step': ([ctypes.POINTER(_CProblem)] + [_P] * 14, ctypes.c_int),
    'hweno_health': ([ctypes.POINTER(_CProblem), _P, _P, ctypes.c_int32], ctypes.c_int),
}
EXPORTS = tuple(_SIGS)

_lib = None


def load_library(path=LIB_PATH):
    """Load libhweno.so (ctypes) and declare its signatures."""
    global _lib
    if _lib is None:
        if not os.path.exists(path):
            raise RuntimeError(f'{path} is missing: build it with '
                               '`python -m paper_2411_11229_amd.build` (no CPU fallback exists)')
        lib = ctypes.CDLL(path)
        for name, (args, res) in _SIGS.items():
            fn = getattr(lib, name)
            fn.argtypes = args
            fn.restype = res
        _lib = lib
    return _lib


def set_strip_rows(rows):
    """Force the strip height of the 2D forward stage kernels (0: automatic);
    results do not depend on it. Process-wide."""
    _check(load_library().hweno_set_strip_rows(int(rows)), 'hweno_set_strip_rows')


def _check(code, what):
    if code != 0:
        raise HwenoError(code, what)


@dataclass
class Problem:
    """Mirror of ``hweno_problem``. gamma0 defaults to 0.95 (1D) / 0.99 (2D)."""
    dim: int
    nx: int
    dx: float
    system: str
    ny: int = 1
    dy: float = 1.0
    adv_a: float = 1.0
    adv_b: float = 1.0
    gas_gamma: float = 1.4
    gamma0: float = None
    d0: float = 0.9
    eps: float = 1e-10
    bc: tuple = ('periodic',) * 4
    precision: str = 'f64'
    basis: str = 'cell'               # characteristic basis: 'cell' | 'interface'
    bc_state: tuple = (None, None, None, None)   # conserved states of 'dirichlet' sides
    gravity: float = 0.0              # g of the (euler2d-s) source, 2D Euler only
    split: tuple = (None, None)       # y_lo / y_hi split rules: dict(x0, slope, speed, kinds, states)

    def __post_init__(self):
        if self.gamma0 is None:
            self.gamma0 = 0.95 if self.dim == 1 else 0.99

    @property
    def ncomp(self):
        return (self.dim + 2) if self.system == 'euler' else 1

    @property
    def dtype(self):
        return torch.float64 if self.precision == 'f64' else torch.float32

    @property
    def shape(self):
        return (self.ncomp, self.nx) if self.dim == 1 else (self.ncomp, self.ny, self.nx)

    def c(self):
        p = _CProblem()
        p.dim, p.nx, p.ny = self.dim, self.nx, self.ny
        p.dx, p.dy = self.dx, self.dy
        p.system = SYSTEMS[self.system]
        p.adv_a, p.adv_b, p.gas_gamma = self.adv_a, self.adv_b, self.gas_gamma
        p.gamma0, p.d0, p.eps = self.gamma0, self.d0, self.eps
        for k in range(4):
            p.bc[k] = BCS[self.bc[k]]
        p.precision = PRECISIONS[self.precision]
        p.char_basis = BASES[self.basis]
        for k, st in enumerate(self.bc_state):
            if st is not None:
                for c, v in enumerate(st):
                    p.bc_state[k][c] = float(v)
        p.gravity = float(self.gravity)
        for k, sp in enumerate(self.split):
            if sp is None:
                continue
            c = p.split[k]
            c.x0, c.slope, c.speed = sp['x0'], sp['slope'], sp['speed']
            for j in range(2):
                c.kind[j] = BCS[sp['kinds'][j]]
                st = (sp.get('states') or (None, None))[j]
                if st is not None:
                    for q, v in enumerate(st):
                        c.state[j][q] = float(v)
        return p


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream(device):
    # the raw handle: torch.cuda.current_stream builds a Stream object (1.5 us),
    # and would refuse other devices itself
    if device.type != 'cuda':
        raise ValueError(f'{device} is not a HIP device')
    index = device.index if device.index is not None else torch.cuda.current_device()
    return ctypes.c_void_p(torch._C._cuda_getCurrentRawStream(index))


class Solver:
    """One problem plus its device workspace (allocated once by torch)."""

    def __init__(self, prob, device='cuda'):
        self.prob = prob
        self.lib = load_library()
        self.cp = _CProblem()
        self.cp = prob.c()
        self.device = torch.device(device)
        self._shape, self._dtype = torch.Size(prob.shape), prob.dtype
        self._made_for = (prob.dim, prob.nx, prob.ny, prob.system, prob.precision)
        nbytes = ctypes.c_size_t()
        _check(self.lib.hweno_workspace_bytes(ctypes.byref(self.cp), ctypes.byref(nbytes)),
               'hweno_workspace_bytes')
        self.ws = torch.empty(nbytes.value, dtype=torch.uint8, device=self.device)
        _check(self.lib.hweno_workspace_init(ctypes.byref(self.cp), _ptr(self.ws),
                                             _stream(self.device)), 'hweno_workspace_init')

    # ------------------------------------------------------------ checks
    def _two(self):
        """Whether the problem is 2D. Every entry point asks first: the arrays are
        checked against, and allocated for, the problem the library was given."""
        p = self.prob
        if (p.dim, p.nx, p.ny, p.system, p.precision) != self._made_for:
            raise ValueError('the problem was changed after its solver was made')
        return p.dim == 2

    def _state(self, t, name, allow_none=False):
        if t is None:
            if allow_none:
                return None
            raise ValueError(f'{name} is required')
        if not isinstance(t, torch.Tensor) or not t.is_cuda:
            raise ValueError(f'{name} must be a HIP-device torch tensor')
        if t.dtype != self._dtype:
            raise ValueError(f'{name}: dtype {t.dtype} != {self.prob.dtype}')
        if t.shape != self._shape:
            raise ValueError(f'{name}: shape {tuple(t.shape)} != {self.prob.shape}')
        if not t.is_contiguous():
            raise ValueError(f'{name} must be contiguous')
        return t

    def _alpha(self, a, name='alpha'):
        if not (isinstance(a, torch.Tensor) and a.dtype == torch.float64 and a.numel() >= 2
                and a.device.type == 'cuda' and a.is_contiguous()):
            raise ValueError(f'{name} must be a contiguous float64 device tensor of 2 values')
        return a

    def new_state(self):
        return torch.empty(self.prob.shape, dtype=self.prob.dtype, device=self.device)

    # ------------------------------------------------------------ entry points
    def max_wavespeed(self, U, out=None):
        self._two()
        U = self._state(U, 'U')
        out = torch.empty(2, dtype=torch.float64, device=self.device) if out is None else out
        _check(self.lib.hweno_max_wavespeed(ctypes.byref(self.cp), _ptr(U), _ptr(self._alpha(out)),
                                            _ptr(self.ws), _stream(self.device)),
               'hweno_max_wavespeed')
        return out

    def rhs(self, U, V, W=None, alpha=None):
        """(L1, L2, L3, vtilde, wtilde); L3, wtilde are None in 1D."""
        two = self._two()
        U, V = self._state(U, 'U'), self._state(V, 'V')
        W = self._state(W, 'W') if two else None
        alpha = self.max_wavespeed(U) if alpha is None else self._alpha(alpha)
        L1, L2, vt = self.new_state(), self.new_state(), self.new_state()
        L3 = self.new_state() if two else None
        wt = self.new_state() if two else None
        _check(self.lib.hweno_rhs(ctypes.byref(self.cp), _ptr(U), _ptr(V), _ptr(W), _ptr(alpha),
                                  _ptr(L1), _ptr(L2), _ptr(L3), _ptr(vt), _ptr(wt), _ptr(self.ws),
                                  _stream(self.device)), 'hweno_rhs')
        return L1, L2, L3, vt, wt

    def step(self, U, V, W, t, t_end=float('inf'), rule='production', cfl=0.6, dt_fixed=0.0,
             dt_used=None, alpha_rec=None, stages=None, events=None):
        """One SSP-RK3 step in place. ``t``: float64 device tensor (in/out).
        ``events``: optional ctypes array of 4 hipEvent_t recorded around the
        three stage launches (hweno_step_profiled)."""
        two = self._two()
        U, V = self._state(U, 'U'), self._state(V, 'V')
        W = self._state(W, 'W') if two else None
        for name, x, n in (('t', t, 1), ('dt_used', dt_used, 1), ('alpha_rec', alpha_rec, 6)):
            if x is not None and not (x.dtype == torch.float64 and x.device.type == 'cuda'
                                      and x.numel() >= n and x.is_contiguous()):
                raise ValueError(f'{name} must be a contiguous float64 device tensor')
        if stages is not None:
            nf = 3 if two else 2
            need = 2 * nf * self.prob.ncomp * self.prob.nx * self.prob.ny
            if not (stages.dtype == self.prob.dtype and stages.numel() >= need
                    and stages.is_contiguous() and stages.device.type == 'cuda'):
                raise ValueError('stages: wrong dtype, size or layout')
        args = (ctypes.byref(self.cp), _ptr(U), _ptr(V), _ptr(W), DT_RULES[rule], float(cfl),
                float(dt_fixed), float(t_end), _ptr(t), _ptr(dt_used), _ptr(alpha_rec),
                _ptr(stages), _ptr(self.ws), _stream(self.device))
        if events is None:
            _check(self.lib.hweno_step(*args), 'hweno_step')
        else:
            _check(self.lib.hweno_step_profiled(*args, events), 'hweno_step_profiled')

    def steps(self, U, V, W, t, nsteps, t_end=float('inf'), rule='production', cfl=0.6,
              dt_fixed=0.0, dt_used=None, alpha_rec=None, events=None):
        """``nsteps`` SSP-RK3 steps in place (hweno_steps): the stage-1 alphas
        of every step after the first come from the previous step's last
        stage. ``dt_used`` / ``alpha_rec``: optional float64 device tensors of
        nsteps / nsteps x 6 values; ``events``: optional ctypes array of
        4 * nsteps hipEvent_t."""
        two = self._two()
        U, V = self._state(U, 'U'), self._state(V, 'V')
        W = self._state(W, 'W') if two else None
        nsteps = int(nsteps)
        for name, x, n in (('t', t, 1), ('dt_used', dt_used, nsteps),
                           ('alpha_rec', alpha_rec, 6 * nsteps)):
            if x is not None and not (x.dtype == torch.float64 and x.device.type == 'cuda'
                                      and x.numel() >= n and x.is_contiguous()):
                raise ValueError(f'{name} must be a contiguous float64 device tensor of {n} values')
        _check(self.lib.hweno_steps(ctypes.byref(self.cp), _ptr(U), _ptr(V), _ptr(W), nsteps,
                                    DT_RULES[rule], float(cfl), float(dt_fixed), float(t_end),
                                    _ptr(t), _ptr(dt_used), _ptr(alpha_rec), _ptr(self.ws),
                                    _stream(self.device), events), 'hweno_steps')

    def _stages_ok(self, stages):
        if stages is None:
            return None
        nf = 3 if self.prob.dim == 2 else 2
        need = 2 * nf * self.prob.ncomp * self.prob.nx * self.prob.ny
        if not (isinstance(stages, torch.Tensor) and stages.dtype == self.prob.dtype
                and stages.numel() >= need and stages.is_contiguous()
                and stages.device.type == 'cuda'):
            raise ValueError('stages: wrong dtype, size or layout')
        return stages

    def _scalars_ok(self, dt, alpha_rec):
        for name, x, n in (('dt', dt, 1), ('alpha_rec', alpha_rec, 6)):
            if not (isinstance(x, torch.Tensor) and x.dtype == torch.float64 and x.numel() >= n
                    and x.is_contiguous() and x.device.type == 'cuda'):
                raise ValueError(f'{name} must be a contiguous float64 device tensor')

    def step_frozen(self, U, V, W, dt, alpha_rec, stages=None, out=None):
        """One step with the given dt (device, 1 value) and stage alphas
        (device, 6 values): the map the adjoint differentiates. In place, or
        into ``out`` = (U', V'[, W']) leaving (U, V, W) unchanged."""
        two = self._two()
        U, V = self._state(U, 'U'), self._state(V, 'V')
        W = self._state(W, 'W') if two else None
        self._scalars_ok(dt, alpha_rec)
        o = [None, None, None]
        if out is not None:
            if len(out) != (3 if two else 2):
                raise ValueError('out: one tensor per field')
            o = [self._state(x, 'out') for x in out] + ([None] if not two else [])
        _check(self.lib.hweno_step_frozen(ctypes.byref(self.cp), _ptr(U), _ptr(V), _ptr(W),
                                          _ptr(o[0]), _ptr(o[1]), _ptr(o[2]), _ptr(dt),
                                          _ptr(alpha_rec), _ptr(self._stages_ok(stages)),
                                          _ptr(self.ws), _stream(self.device)), 'hweno_step_frozen')

    def adjoint_step(self, U, V, W, dt, alpha_rec, lam_in, lam_out, stages=None):
        """dJ/dX^n into ``lam_out`` (3-tuple, or 2-tuple in 1D) from dJ/dX^{n+1}."""
        two = self._two()
        U, V = self._state(U, 'U'), self._state(V, 'V')
        W = self._state(W, 'W') if two else None
        self._scalars_ok(dt, alpha_rec)
        nf = 3 if two else 2
        li = [self._state(x, 'lam_in') for x in list(lam_in)[:nf]] + [None] * (3 - nf)
        lo = [self._state(x, 'lam_out') for x in list(lam_out)[:nf]] + [None] * (3 - nf)
        stages = self._stages_ok(stages)
        _check(self.lib.hweno_adjoint_step(
            ctypes.byref(self.cp), _ptr(U), _ptr(V), _ptr(W if two else None), _ptr(stages),
            _ptr(dt), _ptr(alpha_rec), _ptr(li[0]), _ptr(li[1]), _ptr(li[2] if two else None),
            _ptr(lo[0]), _ptr(lo[1]), _ptr(lo[2] if two else None), _ptr(self.ws),
            _stream(self.device)), 'hweno_adjoint_step')

    def health(self, clear=False):
        """Sync the stream; raise HwenoError if a non-finite / non-physical
        state was flagged since the last clear."""
        _check(self.lib.hweno_health(ctypes.byref(self.cp), _ptr(self.ws), _stream(self.device),
                                     1 if clear else 0), 'state check')

    def run(self, U, V, W, t_end, rule='production', cfl=0.6, max_steps=None, chunk=32,
            record=False, graph=False):
        """Advance in place to t_end (or max_steps). Steps are launched in
        chunks; the device skips steps once t reaches t_end. Returns
        (steps, t, dts[, alpha_recs]) with dts / alphas as device tensors.

        Each chunk is one hweno_steps call: a seeding launch, then the three
        stage kernels per step (a short 1D line in FP64: one launch for up to
        64 steps). graph=True captures one chunk as a HIP
        graph and replays it (one graph launch per chunk): for sizes where
        launch overhead, not the kernels, sets the pace. The results are the
        same bit for bit."""
        t = torch.zeros(1, dtype=torch.float64, device=self.device)
        cap = max_steps if max_steps is not None else 1 << 30
        dts, recs = [], []
        n = 0
        g = None
        if graph and cap >= chunk:
            # one step on copies first: the launch code's one-time queries
            # (occupancy) then stay out of the capture
            c = lambda x: None if x is None else x.clone()
            self.steps(c(U), c(V), c(W), c(t), 1, t_end, rule, cfl)
            gbuf = torch.zeros(chunk, dtype=torch.float64, device=self.device)
            grec = torch.zeros(chunk, 6, dtype=torch.float64, device=self.device) if record else None
            torch.cuda.synchronize(self.device)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                self.steps(U, V, W, t, chunk, t_end, rule, cfl, dt_used=gbuf, alpha_rec=grec)
        while n < cap:
            k = min(chunk, cap - n)
            if g is not None and k == chunk:
                gbuf.zero_()
                g.replay()
                buf = gbuf.clone()
                rec = grec.clone() if record else None
            else:
                buf = torch.zeros(k, dtype=torch.float64, device=self.device)
                rec = torch.zeros(k, 6, dtype=torch.float64, device=self.device) if record else None
                self.steps(U, V, W, t, k, t_end, rule, cfl, dt_used=buf, alpha_rec=rec)
            dts.append(buf)
            if record:
                recs.append(rec)
            n += k
            if float(t.item()) >= t_end:
                break
        dts = torch.cat(dts)
        steps = int((dts > 0).sum().item())
        out = (steps, float(t.item()), dts[:steps])
        if record:
            out = out + (torch.cat(recs)[:steps],)
        return out
