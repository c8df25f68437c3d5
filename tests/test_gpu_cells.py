"""Small contexts run the stage one thread per cell, others (and any context
whose tile or launch is set) by marching workgroups.  Both give the same bits:
the right-hand side, steps with the Courant dt taken on the device, and the
dt itself, over the sizes, boundaries and terms that the cell-parallel path
takes; the call without allocations falls back to the march where only its
arrays fit the static scratch."""
import math

import pytest
import torch

from paper_2405_02483_amd import inputs

pytestmark = pytest.mark.gpu

STRETCH = (0.35, -0.2)
SHAPES = {"min6": (6, 6, 6, False, None), "rows": (7, 37, 11, False, None), "block": (33, 9, 17, False, None),
          "wall_min": (6, 9, 6, True, None), "wall": (20, 22, 24, True, None), "stretched": (9, 8, 14, True, STRETCH)}
EXTRA = dict(e_cool=1.5, t_cool=0.1, rho_cool=math.exp(-2.0), cool_cut=1, omega=(0.3, 0.5, 0.8), c_divb=0.05, c1=0.3)


def _terms(mode):
    from paper_2405_02483_amd import lib
    if mode == "options":
        return dict(EXTRA, terms=lib.T_ALL | lib.T_COOL | lib.T_CORI | lib.T_EDIFFAV | lib.T_LNP | lib.T_DIVB | lib.T_MAX5)
    return dict(nu_const=2e-3, eta_const=1e-3, c1=0.2) if mode == "constant" else {}


def _state(nx, ny, nz, wall, stretch):
    f, box, prm = inputs.stratified(nx, ny, nz, seed=6, noise=0.05, beta_mid=2.0, stretch=stretch)
    if not wall:
        g = box["ngz"]
        f = [a[g:g + nz].copy() for a in f]
        box = dict(box, ngz=0, wall=False)
    return f, box, prm


def _both(ctx, fd):
    got = []
    for march in (False, True):
        if march:
            ctx.set_launch("32x8", 0)
        x = [t.clone() for t in fd]
        F = [t.clone() for t in ctx.rhs(x)]
        ctx.step(x, 0.0, 2)
        got.append(F + [t.clone() for t in x] + [torch.tensor(ctx.last_dt())])
    return got


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("mode", ["core", "options", "constant"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_same_bits_as_the_march(shape, mode, dtype):
    from paper_2405_02483_amd.lib import Context
    f, box, prm = _state(*SHAPES[shape])
    ctx = Context(box, dict(prm, **_terms(mode)), dtype=dtype)
    a, b = _both(ctx, ctx.upload([f]))
    ctx.close()
    for v, (p, q) in enumerate(zip(a, b)):
        assert torch.equal(p.cpu(), q.cpu()), v


def test_ensemble_and_static_scratch():
    from paper_2405_02483_amd.lib import Context
    cases = [_state(*SHAPES[k]) for k in sorted(SHAPES)]
    ctx = Context([c[1] for c in cases], cases[0][2], dtype=torch.float64)
    a, b = _both(ctx, ctx.upload([c[0] for c in cases]))
    ctx.close()
    assert all(torch.equal(p.cpu(), q.cpu()) for p, q in zip(a, b))
    # 210000 float64 cells: 34 arrays fit the 64 MiB, 44 do not
    f, box, prm = inputs.turbulent(n=60, seed=4)
    f = [t[:58] for t in f]
    box = dict(box, nz=58, Lz=58 / 60)
    ctx = Context(box, prm, dtype=torch.float64)
    fd = ctx.upload([f])
    want = [t.clone() for t in ctx.rhs(fd)]
    got = ctx.rhs_noalloc(fd, ctx.empty())
    assert all(torch.equal(p, q) for p, q in zip(want, got))
    ctx.close()
