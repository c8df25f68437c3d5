"""The marching stage on boxes that run one thread per cell by themselves:
every term alone and sets of them, in several tiles and both launch modes, bit
for bit against the cell-parallel stage (which the single-term, closed-form
and wave tests hold against the oracle); chunks of one plane against long ones
in contexts that both march; and a persistent ensemble against the oracle."""
import math
import random

import pytest
import torch

import oracle as O
from paper_2405_02483_amd import inputs
from tests.helpers import grid_params, rel_errors, to_cpu64

pytestmark = pytest.mark.gpu

EXTRA = dict(e_cool=1.5, t_cool=0.1, rho_cool=math.exp(-2.0), cool_cut=1, omega=(0.3, 0.5, 0.8), c_divb=0.05,
             c_smag=0.15, q_max=8.0, q_lim=2.0, d2_lim=0.2, c1=0.3)
MARCH_ONLY = O.T_SMAG | O.T_QUENCH | O.T_ORDER2      # terms the cell-parallel stage lacks
RNG = random.Random(7)
MASKS = ([1 << b for b in range(18) if not (1 << b) & MARCH_ONLY] + [O.T_ALL & ~(1 << b) for b in range(9)] +
         [RNG.randrange(1, 1 << 18) & ~MARCH_ONLY for _ in range(10)] +
         [O.T_PRES | O.T_LNP, O.T_EDIFF | O.T_EDIFFAV, O.T_EDIFF | O.T_MAX5, O.T_VISC | O.T_MAX5, 0])
LAUNCHES = [("32x8", 0, "64x4"), ("16x16", 1, "16x16"), ("16x8", 0, "32x16"), ("64x8", 1, "32x8")]


def _state(nx, ny, nz, wall, stretch=None):
    f, box, prm = inputs.stratified(nx, ny, nz, seed=6, noise=0.05, beta_mid=2.0, stretch=stretch)
    if not wall:
        g = box["ngz"]
        f = [a[g:g + nz].copy() for a in f]
        box = dict(box, ngz=0, wall=False)
    return f, box, prm


def _results(ctx, fd):
    x = [t.clone() for t in fd]
    F = [t.clone() for t in ctx.rhs(x)]
    ctx.step(x, 0.0, 1)
    return F + x + [torch.tensor(ctx.last_dt())]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("kind", ["periodic", "wall", "stretched"])
def test_terms_against_the_cells(kind, dtype):
    from paper_2405_02483_amd.lib import Context
    f, box, prm = _state(19, 11, 13, kind != "periodic", (0.35, -0.2) if kind == "stretched" else None)
    for n, mask in enumerate(MASKS):
        const = dict(nu_const=2e-3, eta_const=1e-3) if n % 3 == 2 else {}
        ctx = Context(box, dict(prm, **dict(EXTRA, terms=mask, **const)), dtype=dtype)
        fd = ctx.upload([f])
        assert ctx.get_cells() == 1
        want = _results(ctx, fd)
        tile, mode, ftile = LAUNCHES[n % len(LAUNCHES)]
        ctx.set_launch(tile, mode)
        ctx.set_final_tile(ftile)
        assert ctx.get_cells() == 0
        for v, (a, b) in enumerate(zip(want, _results(ctx, fd))):
            assert torch.equal(a.cpu(), b.cpu()), (hex(mask), v)
        ctx.close()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("tile", ["32x8", "64x8", "16x16"])
@pytest.mark.parametrize("shape", [(6, 6, 6), (17, 9, 41), (65, 33, 20)])
@pytest.mark.parametrize("wall", [False, True])
def test_short_and_long_chunks(shape, wall, tile, dtype):
    """A box alone has a few dozen tiles' planes for the device, so that the
    cheapest chunk is one plane; among 300 the chunks are longer.  Core terms,
    and every optional term (the Smagorinsky, roughness and quench passes
    march in these chunks too)."""
    from paper_2405_02483_amd.lib import Context
    f, box, prm = _state(*shape, wall)
    for over in ({}, dict(EXTRA, terms=(1 << 18) - 1)):
        got = []
        for copies in (1, 300):
            ctx = Context([box] * copies, dict(prm, **over), dtype=dtype)
            ctx.set_launch(tile, 0)
            fd = ctx.upload([f] * copies)
            F = ctx.rhs(fd)
            first = [t.clone() for t in ctx.box_view(F, 0)]
            assert all(torch.equal(a, b) for a, b in zip(first, ctx.box_view(F, copies - 1)))
            x = [t.clone() for t in fd]
            ctx.step(x, 0.0, 1)
            st = ctx.reductions(fd, F)
            got.append(first + [t.clone() for t in ctx.box_view(x, copies - 1)] +
                       [torch.tensor([ctx.last_dt(), st["dt"], st["cmax"], st["numax"], st["divb_max"]])])
            ctx.close()
        for v, (a, b) in enumerate(zip(*got)):
            assert torch.equal(a.cpu(), b.cpu()), v


@pytest.mark.parametrize("tile,ftile", [("32x8", "32x8"), ("16x16", "64x4"), ("64x8", "32x16")])
def test_persistent_march_of_an_ensemble_matches_oracle(tile, ftile):
    from paper_2405_02483_amd.lib import Context
    sizes = inputs.ensemble_sizes(8, (6, 8, 10, 12), seed=5)
    cases = [inputs.turbulent(n=n, seed=5000 + b, kmax=2.0) for b, n in enumerate(sizes)]
    prm = cases[0][2]
    ctx = Context([c[1] for c in cases], prm, dtype=torch.float32)
    ctx.set_launch(tile, 1)
    ctx.set_final_tile(ftile)
    dt = 0.5 * min(O.courant(to_cpu64(f), *grid_params(b, prm))[0] for f, b, _ in cases)
    fd = ctx.upload([c[0] for c in cases])
    ctx.step(fd, dt, 1)
    assert ctx.get_cells() == 0
    for b, (f, box, _) in enumerate(cases):
        want = O.step(to_cpu64(f), *grid_params(box, prm), dt, 1)
        errs = rel_errors(ctx.box_view(fd, b), want)
        assert max(errs) < 1e-5, (b, sizes[b], errs)
    ctx.close()
