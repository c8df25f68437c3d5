"""The fused transpose of the right-hand side at the sizes where its
addressing changes form: the smallest periodic box (every stencil wraps), rows
that do not fill a workgroup, the shallowest walled boxes (every plane next to
an end) and a stretched one, each with the core terms, all optional terms and
constant coefficients; boxes of every kind in one context.  Float64 against
the oracle's autograd adjoint, 1e-10 relative L2 per field (the bound of the
adjoint's other tests)."""
import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_2405_02483_amd import inputs
from tests.helpers import grid_params, rel_errors, to_cpu64

pytestmark = pytest.mark.gpu

TOL = 1e-10
OPTIONS = dict(terms=O.T_ALL | O.T_COOL | O.T_CORI | O.T_EDIFFAV | O.T_LNP | O.T_DIVB | O.T_SMAG | O.T_MAX5
               | O.T_QUENCH | O.T_ORDER2, e_cool=1.5, t_cool=0.1, rho_cool=math.exp(-2.0), cool_cut=2,
               omega=(0.3, 0.5, 0.8), c_divb=0.05, c_smag=0.15, q_max=8.0, q_lim=2.0, d2_lim=0.2, c1=0.3)
MODES = {"core": {}, "options": OPTIONS, "constant": dict(nu_const=2e-3, eta_const=1e-3, c1=0.2)}


def _noisy(nx, ny, nz, wall, stretch=None, seed=5):
    f, box, prm = inputs.stratified(nx, ny, nz, seed=seed, noise=0.05, beta_mid=2.0, stretch=stretch)
    rng = np.random.default_rng(seed + 1)
    f[0] = f[0] * np.exp(0.05 * rng.standard_normal(f[0].shape))
    f[4] = f[4] * np.exp(0.05 * rng.standard_normal(f[4].shape))
    for v in (5, 6, 7):
        f[v] = f[v] + 0.1 * rng.standard_normal(f[v].shape)
    if not wall:
        g = box["ngz"]
        f = [a[g:g + nz].copy() for a in f]
        box = dict(box, ngz=0, wall=False)
    return f, box, prm


KINDS = {"min6": (6, 6, 6, False, None), "rows": (7, 37, 11, False, None), "flat": (65, 6, 7, False, None),
         "wall_min": (6, 9, 6, True, None), "wall_rows": (33, 7, 13, True, None),
         "stretched": (9, 8, 14, True, (0.35, -0.2))}


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_step_and_rhs_adjoint(kind, mode):
    from paper_2405_02483_amd.lib import Context
    f, box, prm = _noisy(*KINDS[kind])
    g, p = grid_params(box, prm, **MODES[mode])
    ft = to_cpu64(f)
    dt = 0.2 * O.courant(ft, g, p)[0]
    rng = np.random.default_rng(9)
    w = [rng.standard_normal(a.shape) for a in f]
    ctx = Context(box, dict(prm, **MODES[mode]), dtype=torch.float64)
    fd, wd = ctx.upload([f]), ctx.upload([w])
    got = [t.clone() for t in ctx.box_view(ctx.step_adjoint(fd, dt, wd), 0)]
    errs = rel_errors(got, O.step_vjp(ft, g, p, dt, to_cpu64(w)))
    assert max(errs) < TOL, errs
    # the right-hand side alone, fill included
    got = [t.clone() for t in ctx.box_view(ctx.rhs_adjoint(fd, wd), 0)]
    x = tuple(t.clone().requires_grad_(True) for t in ft)
    want = torch.autograd.grad(O.rhs(x, g, p), x, grad_outputs=to_cpu64(w), allow_unused=True)
    errs = rel_errors(got, [torch.zeros_like(a) if b is None else b for a, b in zip(ft, want)])
    ctx.close()
    assert max(errs) < TOL, errs


def test_every_kind_in_one_context():
    from paper_2405_02483_amd.lib import Context
    cases = [_noisy(*KINDS[k], seed=20 + n) for n, k in enumerate(sorted(KINDS))]
    prm = dict(cases[0][2], **OPTIONS)
    dt = 1e-3
    ctx = Context([c[1] for c in cases], prm, dtype=torch.float64)
    rng = np.random.default_rng(3)
    ws = [[rng.standard_normal(a.shape) for a in c[0]] for c in cases]
    out = ctx.step_adjoint(ctx.upload([c[0] for c in cases]), dt, ctx.upload(ws))
    for b, (f, box, _) in enumerate(cases):
        g, p = grid_params(box, cases[0][2], **OPTIONS)
        errs = rel_errors(ctx.box_view(out, b), O.step_vjp(to_cpu64(f), g, p, dt, to_cpu64(ws[b])))
        assert max(errs) < TOL, (box, errs)
    ctx.close()
