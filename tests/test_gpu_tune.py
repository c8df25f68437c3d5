"""mhd_autotune on the GPU: the kept launch is the smallest of the times that
it returns, with one shape or another for pass F, and the results are those of
any launch."""
import pytest
import torch

from paper_2405_02483_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,dtype,boxes", [(12, torch.float32, 6), (12, torch.float64, 1), (32, torch.float64, 1),
                                           (110, torch.float32, 1), (96, torch.float64, 1)])
def test_kept_launch_is_the_fastest(n, dtype, boxes):
    from paper_2405_02483_amd.lib import Context, TILES
    f, box, prm = inputs.turbulent(n=n, seed=8)
    ctx = Context([box] * boxes, prm, dtype=dtype)
    fd = ctx.upload([f] * boxes)
    want = [t.clone() for t in ctx.rhs(fd)]
    for _ in range(3):
        ms = ctx.autotune(fd, reps=2)
        assert len(ms) == 2 * len(TILES) and all(v > 0.0 for v in ms.values())
        assert ctx.get_launch() == min(ms, key=ms.get)
        assert ctx.get_final_tile() in TILES
        for a, b in zip(want, ctx.rhs(fd)):
            assert torch.equal(a, b)
    ctx.close()
