"""div B cleaning over transform lengths: every radix and their products, odd
lengths (rows paired across planes), one row left over, a prime that the
library's own transforms leave to rocFFT, and a mix in one context.  Against
the float64 oracle, with the bounds of the other cleaning tests (1e-12 and
1e-5 relative L2 per component)."""
import numpy as np
import pytest
import torch

import oracle as O
from tests.helpers import rel_errors, to_cpu64

pytestmark = pytest.mark.gpu

PRM = dict(gamma=5.0 / 3.0, mu=1.0)
SHAPES = [(6, 6, 6), (7, 9, 11), (8, 16, 64), (13, 12, 10), (26, 15, 21), (22, 14, 6), (63, 7, 25), (100, 12, 8),
          (128, 6, 30), (250, 6, 7), (6, 208, 8), (9, 6, 256), (17, 8, 12), (12, 38, 6)]


def _fields(shape, seed):
    nx, ny, nz = shape
    rng = np.random.default_rng(seed)
    f = [np.ones((nz, ny, nx)) for _ in range(8)]
    for v in (5, 6, 7):
        f[v] = rng.standard_normal((nz, ny, nx)) + 0.3
    return f, dict(nx=nx, ny=ny, nz=nz, ngz=0, wall=False, Lx=1.1, Ly=0.8, Lz=1.3)


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
def test_lengths(dtype, tol):
    from paper_2405_02483_amd.lib import Context
    cases = [_fields(s, 40 + n) for n, s in enumerate(SHAPES)]
    ctx = Context([c[1] for c in cases], PRM, dtype=dtype)
    fd = ctx.upload([c[0] for c in cases])
    before = [t.clone() for t in fd]
    ctx.divb_clean(fd)
    for b, (f, box) in enumerate(cases):
        want = O.divb_clean(to_cpu64(f), O.Grid(**box))
        errs = rel_errors([t for t in ctx.box_view(fd, b)][5:], want[5:])
        assert max(errs) < tol, (SHAPES[b], errs)
    assert all(torch.equal(p, q) for p, q in zip(before[:5], fd[:5]))
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("shape", [(64, 6, 6), (6, 512, 6), (1024, 6, 6), (6, 6, 720)])
def test_long_axes(shape, dtype):
    from paper_2405_02483_amd.lib import Context
    f, box = _fields(shape, 7)
    ctx = Context(box, PRM, dtype=dtype)
    fd = ctx.upload([f])
    ctx.divb_clean(fd)
    want = O.divb_clean(to_cpu64(f), O.Grid(**box))
    errs = rel_errors(ctx.box_view(fd, 0)[5:], want[5:])
    ctx.close()
    assert max(errs) < (1e-12 if dtype == torch.float64 else 1e-5), errs
