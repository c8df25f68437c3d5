"""The z-chunks of the stage passes follow the size of the whole context: a
box alone (short marches, one plane at the least) and the same box among
many (long ones) give the same bits, and each the oracle's right-hand side."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2405_02483_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", [(6, 6, 6), (17, 9, 41), (65, 33, 20)])
@pytest.mark.parametrize("wall", [False, True])
def test_box_alone_and_among_many(shape, wall, dtype):
    from paper_2405_02483_amd.lib import Context
    nx, ny, nz = shape
    f, box, prm = inputs.stratified(nx, ny, nz, seed=3, noise=0.05, beta_mid=2.0)
    if not wall:     # the interior as a periodic box (the jump at its ends included)
        g = box["ngz"]
        f = [a[g:g + nz].copy() for a in f]
        box = dict(box, ngz=0, wall=False)
    got = []
    for copies in (1, 40):
        ctx = Context([box] * copies, prm, dtype=dtype)
        fd = ctx.upload([f] * copies)
        F = ctx.rhs(fd)
        views = [[t.clone() for t in ctx.box_view(F, b)] for b in (0, copies - 1)]
        for a, b in zip(*views):
            assert torch.equal(a, b)
        got.append(views[0])
        ctx.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)
    if dtype == torch.float64:
        g, p = O.Grid(**box), O.Params(**prm)
        want = O.rhs(tuple(torch.from_numpy(np.ascontiguousarray(a)) for a in f), g, p)
        for v, (a, w) in enumerate(zip(got[0], want)):
            # dp_z is the residual of pressure gradient and gravity: its scale
            scale = float(torch.linalg.norm(w)) + (float(prm["gz"] * torch.linalg.norm(torch.from_numpy(f[0])))
                                                   if v == 3 else 0.0)
            assert float(torch.linalg.norm(a.cpu() - w)) <= 1e-12 * max(scale, 1e-300)
