"""div B cleaning at the sizes where its dispatch changes: above the cells up
to which div B is formed in the x transform (a power of two, and odd lengths
with an odd number of rows), above the cells up to which lengths with odd
factors take the library's own transforms, long x with few rows (few lines a
workgroup), short y and z (many, up to what a workgroup holds).  Each with a small box in the same context,
so that the shared scratch and row pitch are those of the other.  Against the
float64 oracle, with the bounds of the other cleaning tests (1e-12 and 1e-5
relative L2 per component)."""
import time

import numpy as np
import pytest
import torch

import oracle as O
from tests.helpers import rel_errors, to_cpu64

pytestmark = pytest.mark.gpu

PRM = dict(gamma=5.0 / 3.0, mu=1.0)
BIG = [(128, 128, 64), (125, 105, 99), (150, 135, 105)]
LINES = [(500, 9, 20), (512, 9, 6), (1000, 12, 7), (728, 7, 9), (1024, 6, 33), (33, 100, 100), (256, 256, 16),
         (300, 7, 150), (66, 6, 1024), (40, 12, 250),
         # as many lines of a short axis as a workgroup holds of each class
         (256, 512, 11), (128, 1024, 13), (300, 260, 22), (256, 512, 7), (300, 512, 8)]


def _fields(shape, seed):
    nx, ny, nz = shape
    rng = np.random.default_rng(seed)
    f = [np.ones((nz, ny, nx)) for _ in range(8)]
    for v in (5, 6, 7):
        f[v] = rng.standard_normal((nz, ny, nx)) + 0.3
    return f, dict(nx=nx, ny=ny, nz=nz, ngz=0, wall=False, Lx=1.1, Ly=0.8, Lz=1.3)


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
@pytest.mark.parametrize("shape", BIG + LINES)
def test_sizes(shape, dtype, tol):
    from paper_2405_02483_amd.lib import Context
    cases = [_fields((22, 14, 6), 2), _fields(shape, 3), _fields((17, 8, 12), 4)]
    ctx = Context([c[1] for c in cases], PRM, dtype=dtype)
    fd = ctx.upload([c[0] for c in cases])
    for _ in range(2):      # (a clean field stays: the second call's scratch is warm)
        ctx.divb_clean(fd)
    for b, (f, box) in enumerate(cases):
        g = O.Grid(**box)
        want = O.divb_clean(O.divb_clean(to_cpu64(f), g), g)
        errs = rel_errors(ctx.box_view(fd, b)[5:], want[5:])
        assert max(errs) < tol, (b, errs)
    ctx.close()


@pytest.mark.parametrize("n,m", [(500, 20), (512, 32)])
def test_few_long_rows_fill_the_device(n, m):
    """The x transform of a box with few rows takes fewer of them a workgroup:
    a box long in x is no slower than the same long in y (it was 1.4 times
    slower, a quarter of the workgroups)."""
    from paper_2405_02483_amd.lib import Context
    best = []
    for shape in ((n, m, m), (m, n, m)):
        f, box = _fields(shape, 1)
        ctx = Context(box, PRM, dtype=torch.float32)
        fd = ctx.upload([f])
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(50):
                ctx.divb_clean(fd)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        best.append(min(times[1:]))
        ctx.close()
    assert best[0] < 1.2 * best[1], best
