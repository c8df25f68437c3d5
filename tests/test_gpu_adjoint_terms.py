"""The transpose of the right-hand side with part of the terms: every term
alone, all but one, and random sets, with variable and constant coefficients,
between walls and periodic, against the float64 oracle's autograd (1e-10
relative L2 per field, the bound of the adjoint's other tests).  A set of
terms takes the workspace arrays and the passes that it needs: the adjoint of
the continuity alone must not allocate, nor take the time of, the whole
right-hand side's."""
import math
import random
import time

import numpy as np
import pytest
import torch

import oracle as O
from paper_2405_02483_amd import inputs
from tests.helpers import grid_params, rel_errors, to_cpu64

pytestmark = pytest.mark.gpu

TOL = 1e-10
EXTRA = dict(e_cool=1.5, t_cool=0.1, rho_cool=math.exp(-2.0), cool_cut=2, omega=(0.3, 0.5, 0.8), c_divb=0.05,
             c_smag=0.15, q_max=8.0, q_lim=2.0, d2_lim=0.2, c1=0.3)
NBITS = 18
EVERY = (1 << NBITS) - 1
RNG = random.Random(4)
MASKS = ([1 << b for b in range(NBITS)] + [EVERY & ~(1 << b) for b in range(NBITS)] +
         [O.T_ALL & ~(1 << b) for b in range(9)] + [RNG.randrange(1, EVERY) for _ in range(24)] +
         # the terms that only act with another one, each with that one alone
         [O.T_EDIFF | O.T_EDIFFAV, O.T_PRES | O.T_LNP, O.T_EDIFF | O.T_SMAG, O.T_RESIST | O.T_MAX5,
          O.T_VISC | O.T_QUENCH, O.T_VISC | O.T_ORDER2, O.T_RESIST | O.T_SMAG, 0])


def _noisy(nx, ny, nz, wall, seed=5):
    f, box, prm = inputs.stratified(nx, ny, nz, seed=seed, noise=0.05, beta_mid=2.0)
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


@pytest.mark.parametrize("const", [{}, dict(nu_const=2e-3), dict(nu_const=2e-3, eta_const=1e-3), dict(eta_const=1e-3)],
                         ids=["variable", "nu", "nu_eta", "eta"])
@pytest.mark.parametrize("wall", [False, True])
def test_sets_of_terms(wall, const):
    from paper_2405_02483_amd.lib import Context
    f, box, prm = _noisy(7, 6, 8, wall)
    ft = to_cpu64(f)
    w = [np.random.default_rng(9).standard_normal(a.shape) for a in f]
    wt = to_cpu64(w)
    for mask in MASKS:
        over = dict(EXTRA, terms=mask, **const)
        g, p = grid_params(box, prm, **over)
        ctx = Context(box, dict(prm, **over), dtype=torch.float64)
        fd, wd = ctx.upload([f]), ctx.upload([w])
        got = [t.clone() for t in ctx.box_view(ctx.rhs_adjoint(fd, wd), 0)]
        x = tuple(t.clone().requires_grad_(True) for t in ft)
        total = sum((a * b).sum() for a, b in zip(O.rhs(x, g, p), wt)) + sum(0.0 * t.sum() for t in x)
        want = torch.autograd.grad(total, x)
        big = max(float(torch.linalg.norm(t)) for t in want)
        if big == 0.0:
            assert all(float(t.abs().max()) == 0.0 for t in got), hex(mask)
        else:
            errs = rel_errors(got, want)
            assert max(errs) < TOL, (hex(mask), errs)
        # the step's adjoint accumulates the same transposes
        dt = 1e-3
        got = [t.clone() for t in ctx.box_view(ctx.step_adjoint(fd, dt, wd), 0)]
        ctx.close()
        errs = rel_errors(got, O.step_vjp(ft, g, p, dt, wt))
        assert max(errs) < TOL, (hex(mask), "step", errs)


# arrays of the packed field size that one adjoint step took before the
# transpose was fused by hand (an operation-by-operation program): no set of
# terms may take more
ARRAYS = {O.T_CONT: 45, O.T_ADV: 81, O.T_PRES: 54, O.T_LORENTZ: 61, O.T_INDUCT: 73, O.T_COOL: 59, O.T_ALL: 221}


@pytest.mark.parametrize("mask", sorted(ARRAYS))
def test_workspace_follows_the_terms(mask):
    from paper_2405_02483_amd.lib import Context
    f, box, prm = inputs.turbulent(n=96, seed=4)
    ctx = Context(box, dict(prm, **dict(EXTRA, terms=mask)), dtype=torch.float64)
    fd, out = ctx.upload([f]), ctx.empty()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    ctx.step_adjoint(fd, 1e-4, fd, out)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    ctx.close()
    # (one array and 4 MiB for the plane means and the allocator's grain)
    assert used <= (ARRAYS[mask] + 1) * 96 ** 3 * 8 + (4 << 20), used / (96 ** 3 * 8)


def test_time_follows_the_terms():
    """128^3 float32: the transpose of the continuity alone reads the
    cotangents and writes the result; half the whole transpose's time would
    be its passes run for nothing (2.4 times what it took as a program)."""
    from paper_2405_02483_amd.lib import Context
    f, box, prm = inputs.turbulent(n=128, seed=4)
    best = {}
    for mask in (O.T_CONT, O.T_ALL):
        ctx = Context(box, dict(prm, terms=mask), dtype=torch.float32)
        fd, out = ctx.upload([f]), ctx.empty()
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                ctx.rhs_adjoint(fd, fd, out)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        best[mask] = min(times[1:])
        ctx.close()
    assert best[O.T_CONT] < 0.35 * best[O.T_ALL], best
